// P2P of one target leaf against its interaction list (Eq. (8)); shared by the
// single-tree direct route and the batched persistent kernel.
//
// NW wavefronts share one target leaf (sh is private to each wave).  The source
// points of up to 64 list entries at a time form one sequence, cut into chunks of
// 64; the chunks go round the waves.  Within a chunk a block of nt <= 64 targets
// splits the lanes into G = floor(64 / nt) groups of nt (the lanes past G nt idle),
// each group taking every G-th source.  A chunk's partial sums are float32 (at most
// 64 terms) and are added in float64, so the result does not depend on how many
// waves share the leaf (the order of the float64 additions moves it by 2^-53).
// exp(-d^2/sigma^2) is evaluated as exp2(-(k d)^2) with k^2 = log2(e)/sigma^2
// (k = k_scale); the sources of a chunk sit in LDS as one 16-byte record each.
#pragma once
#include "internal.hpp"

namespace msp {
namespace {

struct BoxGeo {
    double lo[3];
    double side;
};

__device__ inline void node_box(const BoxGeo &g, int level, int ix, int iy, int iz, float c[3],
                                float &half) {
    const double h = ldexp(g.side, -level);   // side / 2^level
    c[0] = (float)(g.lo[0] + (ix + 0.5) * h);
    c[1] = (float)(g.lo[1] + (iy + 0.5) * h);
    c[2] = (float)(g.lo[2] + (iz + 0.5) * h);
    half = (float)(0.5 * h);
}

// Interaction lists of a tree's leaves: node v's list is its cnt[v] entries of lst
// from off[v] on, or from v * stride on when stride > 0 (one row per node).
struct LeafLists {
    const int64_t *off;
    int64_t stride;
    const int32_t *cnt, *lst;
    __device__ int64_t begin(int64_t v) const { return stride > 0 ? v * stride : off[v]; }
};

// One tree's arrays as the P2P pass reads them.
struct LeafSet {
    int64_t n_nodes;
    const int32_t *nfirst, *ncount, *nnchild, *nlevel, *nix, *niy, *niz;
    BoxGeo geo;
    LeafLists list;
    const float4 *ps;
    const uint8_t *tflag;
    float k_scale;
    int exclude_self;
    float *usort;
};

// A window of up to 64 list entries: for entry e, the number of source points up to
// and including it, and its first point minus the points before it.
struct ListWindow {
    int32_t efirst[64], incl[64];
};

struct P2PShared {
    // staged sources (scaled offsets from the leaf centre, weight) and their point
    // indices; slots 64..127 hold zero records for the idle lanes' reads
    float4 sp[128];
    int32_t sid[128];
    double red[64];
    ListWindow win;
};

__device__ inline int p2p_incl_scan(int v, int lane) {
    for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(v, o, 64);
        if (lane >= o) v += t;
    }
    return v;
}

// The window's entries w0 .. w0 + 63 of a list of len entries at lst into win;
// returns its source points.  One wavefront; win is written after a wave_sync, so
// the previous window's readers are done.
__device__ inline int load_window(const int32_t *lst, int len, int w0, int64_t n_nodes, const int32_t *nfirst,
                                  const int32_t *ncount, int lane, ListWindow &win) {
    int32_t esf = 0, esn = 0;
    if (w0 + lane < len) {
        const int32_t u = lst[w0 + lane];
        if (u >= 0 && u < n_nodes) {
            esf = nfirst[u];
            esn = ncount[u];
        }
    }
    const int incl = p2p_incl_scan(esn, lane);
    wave_sync();
    win.efirst[lane] = esf - (incl - esn);
    win.incl[lane] = incl;
    wave_sync();
    return __builtin_amdgcn_readfirstlane(__shfl(incl, 63, 64));
}

// Point index of source j of the window (j < its source points): the first entry
// whose inclusive count exceeds j, by six halvings.
__device__ inline int32_t window_point(const ListWindow &win, int j) {
    int e = 0;
#pragma unroll
    for (int st = 32; st > 0; st >>= 1) e = win.incl[e + st - 1] <= j ? e + st : e;
    return win.efirst[e] + j;
}

// Wave `wave` of the NW that share target leaf v; red: one row of 64 per wave (NW > 1).
template <int NW>
__device__ inline void p2p_leaf(const LeafSet &L, int64_t v, int wave, P2PShared &sh, double (*red)[64]) {
    if (v >= L.n_nodes || L.nnchild[v] != 0) return;
    const int lane = threadIdx.x & 63;
    float ct[3], ht;
    node_box(L.geo, L.nlevel[v], L.nix[v], L.niy[v], L.niz[v], ct, ht);
    const int32_t tf = L.nfirst[v], tn = L.ncount[v];
    const int32_t *lst = L.list.lst + L.list.begin(v);
    int len = L.list.cnt[v];
    if (len > L.n_nodes) len = (int)L.n_nodes;   // a list names each node at most once
    sh.sp[64 + lane] = make_float4(0.f, 0.f, 0.f, 0.f);
    sh.sid[64 + lane] = -1;
    for (int t0 = 0; t0 < tn; t0 += 64) {
        const int nt = tn - t0 < 64 ? tn - t0 : 64;
        const int tp = __builtin_amdgcn_readfirstlane(nt);
        const int G = 64 / tp;
        // lane / tp as a multiply by ceil(2^16 / tp): exact for lane < 64, tp <= 64
        const int grp = (lane * ((65536 + tp - 1) / tp)) >> 16;   // grp == G: an idle lane
        const int a = lane - grp * tp;
        const int32_t ti = tf + t0 + a;
        const float4 qt = L.ps[ti];
        const float tx = (qt.x - ct[0]) * L.k_scale;
        const float ty = (qt.y - ct[1]) * L.k_scale;
        const float tz = (qt.z - ct[2]) * L.k_scale;
        double total = 0.0;
        int turn = NW > 1 ? wave : 0;   // this wave's next chunk, counted from the window's first
        for (int w0 = 0; w0 < len; w0 += 64) {
            const int tot = load_window(lst, len, w0, L.n_nodes, L.nfirst, L.ncount, lane, sh.win);
            const int nch = (tot + 63) >> 6;
            float4 nxt = make_float4(0.f, 0.f, 0.f, 0.f);
            int32_t nid = -1;
            // slots past the window's end hold a zero record (weight 0, no point)
            auto fetch = [&](int c) {
                const int j = c * 64 + lane;
                nxt = make_float4(0.f, 0.f, 0.f, 0.f);
                nid = -1;
                if (j < tot) {
                    nid = window_point(sh.win, j);
                    const float4 q = L.ps[nid];
                    nxt = make_float4((q.x - ct[0]) * L.k_scale, (q.y - ct[1]) * L.k_scale,
                                      (q.z - ct[2]) * L.k_scale, q.w);
                }
            };
            if (turn < nch) fetch(turn);
            for (; turn < nch; turn += NW) {
                const int ns = tot - turn * 64 < 64 ? tot - turn * 64 : 64;
                wave_sync();
                sh.sp[lane] = nxt;
                sh.sid[lane] = nid;
                wave_sync();
                // the wave's next chunk is loaded while this one is used
                if (turn + NW < nch) fetch(turn + NW);
                // a group takes sources grp, grp + G, ... of the chunk.  The trip count is the
                // same for every lane (a scalar loop that unrolls); the slots read stay below
                // ns + G <= 128, and a slot past the chunk's end adds exactly 0
                float part = 0.f;
                const int nit = __builtin_amdgcn_readfirstlane((ns + G - 1) / G);
                const float4 *sp = sh.sp + grp;
                const int32_t *sid = sh.sid + grp;
                const int Gs = __builtin_amdgcn_readfirstlane(G);
                if (L.exclude_self) {
#pragma unroll 4
                    for (int it = 0; it < nit; ++it) {
                        const float4 q = sp[it * Gs];
                        const float dx = tx - q.x, dy = ty - q.y, dz = tz - q.z;
                        const float d2 = fmaf(dx, dx, fmaf(dy, dy, dz * dz));
                        const float e = q.w * __builtin_amdgcn_exp2f(-d2);
                        part += sid[it * Gs] == ti ? 0.f : e;
                    }
                } else {
#pragma unroll 4
                    for (int it = 0; it < nit; ++it) {
                        const float4 q = sp[it * Gs];
                        const float dx = tx - q.x, dy = ty - q.y, dz = tz - q.z;
                        const float d2 = fmaf(dx, dx, fmaf(dy, dy, dz * dz));
                        part = fmaf(q.w, __builtin_amdgcn_exp2f(-d2), part);
                    }
                }
                total += (double)part;
            }
            turn -= nch;
        }
        // the groups of a wave in order, then the waves in order
        wave_sync();
        sh.red[lane] = total;
        wave_sync();
        double s = 0.0;
        if (a < nt && grp == 0)
            for (int q = 0; q < G; ++q) s += sh.red[q * tp + a];
        if constexpr (NW > 1) {
            red[wave][lane] = s;
            __syncthreads();
            if (wave == 0 && lane < nt) {
                s = 0.0;
#pragma unroll
                for (int q = 0; q < NW; ++q) s += red[q][lane];
            }
        }
        if (wave == 0 && grp == 0 && a < nt) L.usort[ti] = L.tflag[ti] ? (float)s : 0.f;
        if constexpr (NW > 1) __syncthreads();   // red is free again
    }
}

}  // namespace
}  // namespace msp
