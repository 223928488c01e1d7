// Pieces of the backward pass that the single-tree and the batched kernels share,
// so that both give the same bits: the direct sums with derivatives over the
// interaction list of one target leaf, the evaluation of a cell's Taylor series
// with derivatives at one point, and the combination of a point's two field
// records into its gradients.
//
// Record of a point (kRec floats, key order): the field A of the weights w
// (value, gradient x y z, Laplacian) at offset 0, the field B of the target
// weights g (value, gradient x y z) at offset 5.
#pragma once
#include "p2p_leaf.hpp"

namespace msp {
namespace {

constexpr int kRec = 16;   // floats per point record (64 bytes, one aligned segment)

// One tree's arrays as the direct sums with derivatives read them; the staged
// weights sit in ps.w, records go to out + i * stride (key order i).
struct GradLeafSet {
    int64_t n_nodes;
    const int32_t *nfirst, *ncount, *nnchild, *nlevel, *nix, *niy, *niz;
    BoxGeo geo;
    LeafLists list;
    const float4 *ps;
    float kexp, inv_s2;   // -log2(e) / sigma^2, 1 / sigma^2
    float *out;
};

// One wavefront's staging: sources (offsets from the leaf centre, weight) and their
// second weights; the slots from 64 on hold zeros for the idle lanes' reads.
struct GradShared {
    float4 src[256];
    float sg[256];
    ListWindow win;
};

// What the wavefronts of a leaf share: the ordered running sums in float32, those in
// float64, and whose turn it is to add to either.
struct GradBlock {
    float run[3][64];
    double sum[6][64];
    int turn, turn64;
};
// A wavefront alone needs them when its sources are done: in the place of those.
static_assert(sizeof(GradBlock) <= sizeof(float4) * 256, "the sums fit where the sources were");

// A scalar whose uses stay where they are: the slots' addresses, kept in registers across
// the units, would spill.
__device__ inline int not_hoisted(int x) {
    asm volatile("" : "+s"(x));
    return x;
}

// For every point of the target leaf of task t: the sums over the source leaves of its
// list of e = w exp(-r^2/sigma^2), e (x - s) and e r^2, written as value, gradient and
// Laplacian of the field; TWO: also of a second field with the key-order weights g2 of the
// sources (value and gradient, into out + 5), one exponential serving both.
//
// NW wavefronts share the leaf (sh is private to each, bk common).  A block of nt <= 64
// targets splits the lanes into G = floor(64 / nt) groups of nt (the lanes past G nt
// idle), each group taking every G-th source of a 64-source chunk of a window of 64 list
// entries.  The values and the Laplacian are float32 running sums over the whole list in
// its order, which is a serial chain however many wavefronts share the leaf.  So each
// wavefront evaluates units of at most 16 sources a group (the chunk, or a part of it
// where G < 4), keeps the weights, exp and r^2 of every pair in registers, and adds them
// when its turn comes: four instructions a pair in the chain in place of some 25, and no
// load.  The gradients are float32 per unit and float64 over the units, added in the units'
// order too, in a turn of its own behind the first: a leaf's records have the same bits
// however many wavefronts share it.  5,003 points, both fields:
// 162 us with a wavefront per kind of sum, 72 us with eight per leaf; 48 populations of
// 1,024 to 32,768 points: 1.61 ms with a wavefront per leaf, whose largest leaves were the
// launch's tail, 1.0 ms with four.
template <int NW, bool TWO>
__device__ inline void p2p_grad_leaf(const GradLeafSet &L, const float *g2, const LeafTask &t, int stride, int want_lap,
                                     int wave, GradShared &sh, GradBlock &bk) {
    const int lane = threadIdx.x & 63, len = t.len;
    for (int t0 = 0; t0 < t.count; t0 += 64) {
#pragma unroll
        for (int c = 64; c < 256; c += 64) {
            sh.src[c + lane] = make_float4(0.f, 0.f, 0.f, 0.f);
            sh.sg[c + lane] = 0.f;
        }
        const int nt = __builtin_amdgcn_readfirstlane(t.count - t0 < 64 ? t.count - t0 : 64);
        const int G = __builtin_amdgcn_readfirstlane(64 / nt);
        // lane / nt as a multiply by ceil(2^16 / nt): exact for lane < 64, nt <= 64
        const int grp = (lane * ((65536 + nt - 1) / nt)) >> 16;   // grp == G: an idle lane
        const int a = lane - grp * nt;
        const int32_t ti = t.first + t0 + a;
        const float4 qt = ld_global4(L.ps, a < nt ? ti : t.first);
        const float tx = qt.x - t.ct[0], ty = qt.y - t.ct[1], tz = qt.z - t.ct[2];
        const int unit = G < 4 ? 16 * G : 64;
        float su = 0.f, sr = 0.f, gu = 0.f;
        double total[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
        if constexpr (NW > 1) {
            if (wave == 0) {
                bk.run[0][lane] = bk.run[1][lane] = bk.run[2][lane] = 0.f;
#pragma unroll
                for (int c = 0; c < 6; ++c) bk.sum[c][lane] = 0.0;
                if (lane == 0) bk.turn = bk.turn64 = 0;
            }
            __syncthreads();
        }
        int mine = NW > 1 ? wave : 0;   // this wave's next unit, counted from the window's first
        int before = 0;                 // units of the windows before
        for (int w0 = 0; w0 < len; w0 += 64) {
            int start;
            const int tot = load_window(t.lst, w0, len - w0 < 64 ? len - w0 : 64, L.n_nodes, L.nfirst, L.ncount, lane,
                                        sh.win, start);
            const int units = __builtin_amdgcn_readfirstlane(G == 3 ? 2 * (tot >> 6) + ((tot & 63) + 47) / 48
                                                                    : (tot + unit - 1) / unit);
            // the next unit's points as they lie in memory (nothing waits for them before they
            // are staged); lanes past the unit or the window take a target's, with weights 0
            float4 nxt = make_float4(0.f, 0.f, 0.f, 0.f);
            float ngw = 0.f;
            bool valid = false;
            auto fetch = [&](int u) {
                // (G = 3: units of 48, 16 sources of a chunk of 64)
                const int c = G == 3 ? u >> 1 : (u * unit) >> 6, o = G == 3 ? 48 * (u & 1) : (u * unit) & 63;
                const int32_t pj = window_point(sh.win, start, c, o + lane < 63 ? o + lane : 63);
                valid = lane < unit && o + lane < 64 && c * 64 + o + lane < tot;
                const int32_t i = valid ? pj : t.first;
                nxt = ld_global4(L.ps, i);
                if constexpr (TWO) ngw = ld_global(g2, i);
            };
            if (mine < units) fetch(mine);
            for (; mine < units; mine += NW) {
                const int ns = __popcll(__ballot(valid));
                wave_sync();
                sh.src[lane] = make_float4(nxt.x - t.ct[0], nxt.y - t.ct[1], nxt.z - t.ct[2], valid ? nxt.w : 0.f);
                if constexpr (TWO) sh.sg[lane] = valid ? ngw : 0.f;
                wave_sync();
                if (mine + NW < units) fetch(mine + NW);
                // group grp takes sources grp, grp + G, ...: the same trip count on every lane,
                // in fours; the slots read stay below 3 G + ns + G <= 256 (G = 64) or 128, and a
                // slot past the unit's end adds zeros
                const int nit = __builtin_amdgcn_readfirstlane((ns + G - 1) / G);
                const float4 *src = sh.src + grp;
                const float *sg = sh.sg + grp;
                float ke[16], r2[16];
                float px = 0.f, py = 0.f, pz = 0.f, qx = 0.f, qy = 0.f, qz = 0.f;
#pragma unroll
                for (int b = 0; b < 16; b += 4) {
                    if (b >= nit) continue;
                    const int Gs = not_hoisted(G);
#pragma unroll
                    for (int i = b; i < b + 4; ++i) {
                        const float4 s4 = src[i * Gs];
                        const float dx = tx - s4.x, dy = ty - s4.y, dz = tz - s4.z;
                        r2[i] = fmaf(dx, dx, fmaf(dy, dy, dz * dz));
                        ke[i] = __builtin_amdgcn_exp2f(r2[i] * L.kexp);
                        const float e = s4.w * ke[i];
                        px = fmaf(e, dx, px);
                        py = fmaf(e, dy, py);
                        pz = fmaf(e, dz, pz);
                        if constexpr (TWO) {
                            const float g = sg[i * Gs], eg = g * ke[i];
                            if constexpr (NW == 1) gu = fmaf(g, ke[i], gu);
                            qx = fmaf(eg, dx, qx);
                            qy = fmaf(eg, dy, qy);
                            qz = fmaf(eg, dz, qz);
                        }
                        if constexpr (NW == 1) {
                            sr = fmaf(e, r2[i], sr);
                            su = fmaf(s4.w, ke[i], su);
                        }
                    }
                }
                const float part[6] = {px, py, pz, qx, qy, qz};
                if constexpr (NW == 1) {
#pragma unroll
                    for (int c = 0; c < (TWO ? 6 : 3); ++c) total[c] += (double)part[c];
                    continue;
                }
                // (the weights again, before the turn: they need not be live above)
                float wt[16], gw[16];
#pragma unroll
                for (int b = 0; b < 16; b += 4) {
                    if (b >= nit) continue;
                    const int Gs = not_hoisted(G);
#pragma unroll
                    for (int i = b; i < b + 4; ++i) {
                        wt[i] = src[i * Gs].w;
                        if constexpr (TWO) gw[i] = sg[i * Gs];
                    }
                }
                // the turns come round: every earlier unit belongs to a wave of this block that
                // is at it or will be without waiting for this one
                while (__hip_atomic_load(&bk.turn, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) != before + mine)
                    __builtin_amdgcn_s_sleep(1);
                su = bk.run[0][lane];
                sr = bk.run[1][lane];
                if constexpr (TWO) gu = bk.run[2][lane];
#pragma unroll
                for (int b = 0; b < 16; b += 4) {
                    if (b >= nit) continue;
#pragma unroll
                    for (int i = b; i < b + 4; ++i) {
                        sr = fmaf(wt[i] * ke[i], r2[i], sr);
                        su = fmaf(wt[i], ke[i], su);
                        if constexpr (TWO) gu = fmaf(gw[i], ke[i], gu);
                    }
                }
                bk.run[0][lane] = su;
                bk.run[1][lane] = sr;
                if constexpr (TWO) bk.run[2][lane] = gu;
                __hip_atomic_store(&bk.turn, before + mine + 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
                while (__hip_atomic_load(&bk.turn64, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) != before + mine)
                    __builtin_amdgcn_s_sleep(1);
#pragma unroll
                for (int c = 0; c < (TWO ? 6 : 3); ++c) bk.sum[c][lane] += (double)part[c];
                __hip_atomic_store(&bk.turn64, before + mine + 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
            mine -= units;
            before += units;
        }
        if constexpr (NW > 1) {
            __syncthreads();
        } else {
            wave_sync();   // the sources are no longer read
#pragma unroll
            for (int c = 0; c < (TWO ? 6 : 3); ++c) bk.sum[c][lane] = total[c];
            bk.run[0][lane] = su;
            bk.run[1][lane] = sr;
            bk.run[2][lane] = gu;
            wave_sync();
        }
        if (wave == 0 && grp == 0 && a < nt) {
            float r[3] = {0.f, 0.f, 0.f};
            double v[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
            for (int q = 0; q < G; ++q) {
#pragma unroll
                for (int c = 0; c < 3; ++c) r[c] += bk.run[c][q * nt + a];
#pragma unroll
                for (int c = 0; c < (TWO ? 6 : 3); ++c) v[c] += bk.sum[c][q * nt + a];
            }
            float *o = L.out + (int64_t)ti * stride;   // value, gradient x y z, Laplacian
            const double m2 = -2.0 * (double)L.inv_s2;
            o[0] = r[0];
            o[1] = (float)(m2 * v[0]);
            o[2] = (float)(m2 * v[1]);
            o[3] = (float)(m2 * v[2]);
            if (want_lap) o[4] = 4.f * L.inv_s2 * L.inv_s2 * r[1] - 6.f * L.inv_s2 * r[0];
            if constexpr (TWO) {
                o[5] = r[2];
                o[6] = (float)(m2 * v[3]);
                o[7] = (float)(m2 * v[4]);
                o[8] = (float)(m2 * v[5]);
            }
        }
        if constexpr (NW > 1) __syncthreads();   // the block's sums are free again
        else wave_sync();
    }
}

// The gradients of input point j from its record (rec4: the record as float4),
// its target weight g and weight wj; returns its term of the sigma derivative.
__device__ inline double combine_point(const float4 *rec4, float g, float wj, int want_w, int want_pos,
                                       int want_sigma, double sigma, int exclude_self, float *gw, float *gx,
                                       float *gy, float *gz) {
    const float4 a = rec4[0], b = rec4[1], c = rec4[2];
    // a = (Av, Agx, Agy, Agz), b = (Alap, Bv, Bgx, Bgy), c = (Bgz, -, -, -)
    if (want_w) *gw = exclude_self ? b.y - g : b.y;
    if (want_pos) {
        *gx = g * a.y + wj * b.z;
        *gy = g * a.z + wj * b.w;
        *gz = g * a.w + wj * c.x;
    }
    return want_sigma ? (double)g * (0.5 * sigma * (double)b.x + 3.0 / sigma * (double)a.x) : 0.0;
}

}  // namespace
}  // namespace msp
