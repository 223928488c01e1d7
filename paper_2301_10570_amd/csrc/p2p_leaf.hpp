// P2P of one target leaf against its interaction list (Eq. (8)); shared by the
// single-tree direct route and the batched kernel.
//
// NW wavefronts share one target leaf (sh is private to each wave).  The list is cut
// into windows of at most 64 entries (p2p_window), which go round the waves; the source
// points of a window form one sequence, staged in LDS in chunks of 128.  At most 32 terms
// are added one after another in float32, and in the matrix form sixteen such sums in
// pairs; the rest is float64, so the result does not depend on how many waves share the
// leaf (the order of the float64 additions moves it by 2^-53).  exp(-d^2/sigma^2) is
// evaluated as exp2(-d^2) of coordinates from the leaf centre scaled by k_scale =
// sqrt(log2(e)) / sigma.
//
// Two forms, by the size of the leaf against sigma (see kMatrixReach):
//   p2p_block_matrix   exp2(-d^2) = exp2(-t^2) exp2(2 t.s - s^2): the exponents 2 t.s - s^2 of
//       16 targets and 16 sources come from one matrix instruction, the other factor is one
//       value per target, and a pair costs one exponential and one multiply-add on the
//       vector unit in place of eight instructions.
//   p2p_block_vector   the differences themselves.  T = 1, 2 or 4 targets per lane (nt up
//       to 9, 18, 64), the lanes in G = floor(64 / ceil(nt / T)) groups, each taking
//       every G-th source: nine tenths of the lanes' targets are there (one target per
//       lane: 84%) and a record read from LDS serves T pairs.
//
// The vector unit bounds both.  256 populations of 1,024 to 65,536 points (5.0e9 pairs,
// half of them of leaves of at most 16 points) took 2.15 ms with one target per lane and a
// wavefront per leaf, and take 1.74 ms (of which the sums are half, the rest finds and
// stages the sources).
#pragma once
#include "internal.hpp"

namespace msp {
namespace {

// Loads through pointers that a kernel reads from memory (a batch's descriptors): the
// compiler does not know that they are global and would make flat loads, which wait on
// LDS traffic too.
template <typename T>
__device__ inline T ld_global(const T *p, int64_t i) {
    return reinterpret_cast<const __attribute__((address_space(1))) T *>(reinterpret_cast<uintptr_t>(p))[i];
}
__device__ inline float4 ld_global4(const float4 *p, int64_t i) {
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    const f32x4 v =
        reinterpret_cast<const __attribute__((address_space(1))) f32x4 *>(reinterpret_cast<uintptr_t>(p))[i];
    return make_float4(v.x, v.y, v.z, v.w);
}

// A descriptor that is the same for the whole wavefront, in scalar registers.
template <typename T>
__device__ inline T uniform_copy(const T &from) {
    int32_t w[sizeof(T) / 4];
    __builtin_memcpy(w, &from, sizeof(T));
#pragma unroll
    for (int i = 0; i < (int)(sizeof(T) / 4); ++i) w[i] = __builtin_amdgcn_readfirstlane(w[i]);
    T to;
    __builtin_memcpy(&to, w, sizeof(T));
    return to;
}

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
    __device__ int64_t begin(int64_t v) const { return stride > 0 ? v * stride : ld_global(off, v); }
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

// What a wavefront needs to know of a target leaf before it reads the list: its points,
// its list, its centre and half side.  No points: not a leaf.
struct LeafTask {
    const int32_t *lst;
    int32_t len, first, count, owner;   // owner: which of a batch's descriptors
    float ct[3], half;
};

// Node v of a tree (SET: LeafSet or what the derivatives read).
template <class SET>
__device__ inline LeafTask leaf_task(const SET &L, int64_t v, int owner) {
    LeafTask t{nullptr, 0, 0, 0, owner, {0.f, 0.f, 0.f}, 0.f};
    if (v >= L.n_nodes || L.nnchild[v] != 0) return t;
    node_box(L.geo, L.nlevel[v], L.nix[v], L.niy[v], L.niz[v], t.ct, t.half);
    t.first = L.nfirst[v];
    t.count = L.ncount[v];
    t.lst = L.list.lst + L.list.begin(v);
    t.len = L.list.cnt[v];
    if (t.len > L.n_nodes) t.len = (int)L.n_nodes;   // a list names each node at most once
    return t;
}

// A window of up to 64 list entries as runs of consecutive points (neighbours in key
// order often follow each other): run e's first point less the points of the window
// before it (those stay in registers, lane e: run e).
struct ListWindow {
    int32_t base[64];
};

constexpr int kP2PChunk = 128;   // sources staged at a time
constexpr uint8_t kNoTarget = 255;

struct P2PShared {
    // staged sources and which target of the block each is (kNoTarget: none); 64 slots
    // past them hold zero records for the idle lanes' reads
    float4 sp[kP2PChunk + 64];
    float sw[kP2PChunk];
    double red[64];
    ListWindow win;
    uint8_t sid[kP2PChunk + 64];
};

// Inclusive sum over the wavefront (rows of 16 lanes, then the rows' totals).
__device__ inline int p2p_incl_scan(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);   // row_shr 1, 2, 4, 8
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);   // row_bcast 15, 31
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);
    return v;
}

// The entries first .. first + n - 1 (n <= 64) of the list at lst into win; start: the
// window's points before this lane's run (a value past any point on lanes without one).
// Returns the window's points.  One wavefront; win is written after a wave_sync, so the
// previous window's readers are done.
__device__ inline int load_window(const int32_t *lst, int first, int n, int64_t n_nodes, const int32_t *nfirst,
                                  const int32_t *ncount, int lane, ListWindow &win, int &start) {
    int32_t esf = 0, esn = 0;
    if (lane < n) {
        const int32_t u = ld_global(lst, first + lane);
        if (u >= 0 && u < n_nodes) {
            esf = ld_global(nfirst, u);
            esn = ld_global(ncount, u);
        }
    }
    const int incl = p2p_incl_scan(esn);
    const int32_t before = __shfl_up(esf + esn, 1, 64);
    const bool begins = esn > 0 && (lane == 0 || esf != before);
    const uint64_t runs = __ballot(begins);
    const int e = __popcll(runs & ((1ull << lane) - 1ull));
    wave_sync();
    if (begins) win.base[e] = esf - (incl - esn);
    const int moved = __builtin_amdgcn_ds_permute((begins ? e : 63) * 4, incl - esn);
    start = lane < __popcll(runs) ? moved : 0x7fffffff;
    wave_sync();
    return __builtin_amdgcn_readlane(incl, 63);
}

// Point index of source c * 64 + lane of the window (of no meaning past its points):
// the runs that start inside block c of 64 are marked in a scalar mask (a few lane reads
// in place of six dependent halvings per lane).  The whole wavefront calls it.
__device__ inline int32_t window_point(const ListWindow &win, int start, int c, int lane) {
    const int e0 = __popcll(__ballot(start < c * 64));
    const int e1 = __popcll(__ballot(start < c * 64 + 64));
    if (e0 == e1) return win.base[e0 - 1] + c * 64 + lane;
    uint64_t mark = 0ull;
    for (int e = e0; e < e1; ++e) mark |= 1ull << (__builtin_amdgcn_readlane(start, e) - c * 64);
    // runs that start at or before this lane's source, less one (at least one does)
    const uint64_t upto = mark & (lane < 63 ? (2ull << lane) - 1ull : ~0ull);
    return win.base[e0 + (int)__popcll(upto) - 1] + c * 64 + lane;
}

// Entries per window of a list of len: sixteen windows for the sixteen wavefronts that
// may share a leaf, of 8 to 64 entries.  Trees of more leaves than the chip has wavefront
// slots have a wavefront per leaf, for which windows of 8 are so many more chains of
// dependent loads: 64 entries (40,000 points in leaves of one, lists of some 30: 81 us with
// 64 before the leaves were shared, 254 us with 8).  The rule looks at the tree alone, so that
// a batch's launch, which always shares, cuts a list as the tree's own call does.
__device__ inline int p2p_window(int len, int64_t n_nodes) {
    const int w = (len + 15) >> 4;
    return n_nodes > kSharedNodes ? 64 : w < 8 ? 8 : (w > 64 ? 64 : w);
}

// The wave's walk over its windows and their chunks: stage(nxt, nid, own) puts a chunk's
// points (as they lie in memory) and their indices (-1: none) into sh, lane l holding
// sources l and 64 + l; use(sources, own, flush) forms the sums over it, flush: the
// fourth chunk since the last one or the window's last.  own: the chunk holds
// points of the block tf .. tf + nt - 1 and self pairs are excluded.  The next chunk is
// loaded while one is used: nothing waits for it before it is staged.
template <int NW, class Stage, class Use>
__device__ inline void p2p_sources(const LeafSet &L, const int32_t *lst, int len, int32_t tf, int nt, int wave,
                                   P2PShared &sh, Stage stage, Use use) {
    constexpr int PER = kP2PChunk / 64;
    const int lane = threadIdx.x & 63;
    const int W = __builtin_amdgcn_readfirstlane(p2p_window(len, L.n_nodes));
    for (int w0 = wave * W; w0 < len; w0 += NW * W) {
        int start;
        const int tot = load_window(lst, w0, len - w0 < W ? len - w0 : W, L.n_nodes, L.nfirst, L.ncount, lane, sh.win,
                                    start);
        float4 nxt[PER];
        int32_t nid[PER];
        auto fetch = [&](int c0) {
#pragma unroll
            for (int h = 0; h < PER; ++h) {
                // lanes past the window's end take a target's, with index -1
                nid[h] = -1;
                int32_t i = tf;
                if (c0 + 64 * h < tot) {
                    const int32_t at = window_point(sh.win, start, (c0 >> 6) + h, lane);
                    if (c0 + 64 * h + lane < tot) nid[h] = i = at;
                }
                nxt[h] = ld_global4(L.ps, i);
            }
        };
        if (tot > 0) fetch(0);
        for (int c0 = 0; c0 < tot; c0 += kP2PChunk) {
            bool own = false;
            if (L.exclude_self) {
#pragma unroll
                for (int h = 0; h < PER; ++h) own |= __ballot((unsigned)(nid[h] - tf) < (unsigned)nt) != 0;
            }
            wave_sync();
            stage(nxt, nid);
            if (own) {
#pragma unroll
                for (int h = 0; h < PER; ++h)
                    sh.sid[64 * h + lane] =
                        (unsigned)(nid[h] - tf) < (unsigned)nt ? (uint8_t)(nid[h] - tf) : kNoTarget;
            }
            wave_sync();
            if (c0 + kP2PChunk < tot) fetch(c0 + kP2PChunk);
            use(tot - c0, own, c0 + kP2PChunk >= tot || (c0 / kP2PChunk & 3) == 3);
        }
    }
}

// Targets tf .. tf + nt - 1 (T per lane): this wave's windows of the list, into its share
// of the sums (lane l: target l, for l < nt).
template <int NW, int T>
__device__ inline double p2p_block_vector(const LeafSet &L, const int32_t *lst, int len, const float ct[3], int32_t tf,
                                          int nt, int wave, P2PShared &sh) {
    const int lane = threadIdx.x & 63;
    const int tp = __builtin_amdgcn_readfirstlane((nt + T - 1) / T);
    const int G = __builtin_amdgcn_readfirstlane(64 / tp), nfull = __builtin_amdgcn_readfirstlane((kP2PChunk + G - 1) / G);
    // lane / tp as a multiply by ceil(2^16 / tp): exact for lane < 64, tp <= 64
    const int grp = (lane * ((65536 + tp - 1) / tp)) >> 16;   // grp == G: an idle lane
    const int a = lane - grp * tp;
    float tx[T], ty[T], tz[T];
    double total[T];
#pragma unroll
    for (int k = 0; k < T; ++k) {
        const float4 qt = ld_global4(L.ps, tf + (a + k * tp < nt ? a + k * tp : nt - 1));
        tx[k] = (qt.x - ct[0]) * L.k_scale;
        ty[k] = (qt.y - ct[1]) * L.k_scale;
        tz[k] = (qt.z - ct[2]) * L.k_scale;
        total[k] = 0.0;
    }
    auto stage = [&](const float4 *nxt, const int32_t *nid) {
#pragma unroll
        for (int h = 0; h < kP2PChunk / 64; ++h)
            sh.sp[64 * h + lane] =
                make_float4((nxt[h].x - ct[0]) * L.k_scale, (nxt[h].y - ct[1]) * L.k_scale,
                            (nxt[h].z - ct[2]) * L.k_scale, nid[h] < 0 ? 0.f : nxt[h].w);
    };
    // a group takes sources grp, grp + G, ... of the chunk.  The trip count is the same for
    // every lane (a scalar loop); the slots read stay below the chunk's sources + G, and a
    // slot past them adds exactly 0
    auto use = [&](int left, bool own, bool) {
        float part[T];
#pragma unroll
        for (int k = 0; k < T; ++k) part[k] = 0.f;
        const int nit = left >= kP2PChunk ? nfull : __builtin_amdgcn_readfirstlane((left + G - 1) / G);
        const float4 *sp = sh.sp + grp;
        if (own) {
            const uint8_t *sid = sh.sid + grp;
            for (int it = 0; it < nit; ++it) {
                const float4 q = sp[it * G];
                const int id = sid[it * G];
#pragma unroll
                for (int k = 0; k < T; ++k) {
                    const float dx = tx[k] - q.x, dy = ty[k] - q.y, dz = tz[k] - q.z;
                    const float d2 = fmaf(dx, dx, fmaf(dy, dy, dz * dz));
                    part[k] = fmaf(id == a + k * tp ? 0.f : q.w, __builtin_amdgcn_exp2f(-d2), part[k]);
                }
            }
        } else {
#pragma unroll 4 / T
            for (int it = 0; it < nit; ++it) {
                const float4 q = sp[it * G];
#pragma unroll
                for (int k = 0; k < T; ++k) {
                    const float dx = tx[k] - q.x, dy = ty[k] - q.y, dz = tz[k] - q.z;
                    const float d2 = fmaf(dx, dx, fmaf(dy, dy, dz * dz));
                    part[k] = fmaf(q.w, __builtin_amdgcn_exp2f(-d2), part[k]);
                }
            }
        }
#pragma unroll
        for (int k = 0; k < T; ++k) total[k] += (double)part[k];
    };
    p2p_sources<NW>(L, lst, len, tf, nt, wave, sh, stage, use);
    // the groups of the wave in order; lane l gathers target l = (l / tp) tp + l % tp
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < T; ++k) {
        wave_sync();
        sh.red[lane] = total[k];
        wave_sync();
        if (grp == k)   // T <= G: the group exists
            for (int q = 0; q < G; ++q) s += sh.red[q * tp + a];
    }
    return s;
}

// Largest scaled distance of a target from its leaf's centre for the matrix form, whose
// error grows with the size of 2 t.s and s^2 against d^2.  Measured against float64 over
// 512 leaves of 10 and 40 points, root mean square (largest) relative error of a sum, the
// compensated float32 sums of differences that this replaced -> matrix form: reach 0.3:
// 6.6e-8 (2.0e-7) -> 5.6e-8 (1.5e-7); 0.6: 8.1e-8 (2.3e-7) -> 7.6e-8 (2.3e-7); 1: 8.3e-8
// (3.2e-7) -> 7.9e-8 (2.4e-7); 1.2: 9.2e-8 (3.8e-7) -> 9.1e-8 (2.9e-7), at 10 points 9.0e-8
// -> 9.1e-8; 1.5 at 10 points: 1.14e-7 -> 1.19e-7.  At 1 no figure is larger.
constexpr float kMatrixReach = 1.f;

// 2^x for a small x (|x| below 127; to 1e-11): the nearest whole power, and the Taylor
// series of the rest's exponential.
__device__ inline double exp2_near(double x) {
    const double n = rint(x), y = 0.69314718055994531 * (x - n);
    double e = 1.0;
#pragma unroll
    for (int k = 10; k > 0; --k) e = fma(e, y * (1.0 / k), 1.0);
    return ldexp(e, (int)n);
}

// exp2(-t^2) of point i of the leaf about ct
__device__ inline double target_factor(const LeafSet &L, int32_t i, const float *ct) {
    const float4 q = ld_global4(L.ps, i);
    const double x = (q.x - ct[0]) * L.k_scale, y = (q.y - ct[1]) * L.k_scale, z = (q.z - ct[2]) * L.k_scale;
    return exp2_near(-(x * x + y * y + z * z));
}

template <int CTRL>
__device__ inline float dpp(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, false));
}

// The same by matrix products, M = ceil(nt / 16) tiles of 16 targets; the sums lack the
// factors exp2(-t^2).  Lane l holds of a tile (v_mfma_f32_16x16x4f32): operand A target
// l % 16, operand B source l % 16, both their component l / 16, the fourth being -1 and
// s^2; result source l % 16 and targets 4 (l / 16) .. + 3.  2 t.s - s^2 = t^2 - d^2 is at
// most kMatrixReach^2 and never underflows before -d^2 does, so a weight keeps its range
// (up to 2^127; see p2p_leaf).
template <int NW, int M>
__device__ inline double p2p_block_matrix(const LeafSet &L, const int32_t *lst, int len, const float ct[3], int32_t tf,
                                          int nt, int wave, P2PShared &sh) {
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    const int lane = threadIdx.x & 63, col = lane & 15, comp = lane >> 4;
    float A[M], part[M][4];
    double total[M];   // lane l: target 4 (l / 16) + l % 4 of each tile
#pragma unroll
    for (int m = 0; m < M; ++m) {
        const float4 q = ld_global4(L.ps, tf + (16 * m + col < nt ? 16 * m + col : nt - 1));
        const float c = comp == 0 ? q.x - ct[0] : comp == 1 ? q.y - ct[1] : q.z - ct[2];
        A[m] = comp == 3 ? -1.f : 2.f * (c * L.k_scale);
        total[m] = 0.0;
#pragma unroll
        for (int r = 0; r < 4; ++r) part[m][r] = 0.f;
    }
    auto stage = [&](const float4 *nxt, const int32_t *nid) {
#pragma unroll
        for (int h = 0; h < kP2PChunk / 64; ++h) {
            const float x = (nxt[h].x - ct[0]) * L.k_scale, y = (nxt[h].y - ct[1]) * L.k_scale,
                        z = (nxt[h].z - ct[2]) * L.k_scale;
            sh.sp[64 * h + lane] = make_float4(x, y, z, fmaf(x, x, fmaf(y, y, z * z)));
            sh.sw[64 * h + lane] = nid[h] < 0 ? 0.f : nxt[h].w;
        }
    };
    auto use = [&](int left, bool own, bool flush) {
        const float *B = reinterpret_cast<const float *>(sh.sp) + 4 * col + comp;
        const int n16 = __builtin_amdgcn_readfirstlane(left >= kP2PChunk ? kP2PChunk / 16 : (left + 15) >> 4);
        if (own) {
            for (int g = 0; g < n16; ++g) {
                const float b = B[64 * g], w = sh.sw[16 * g + col];
                const int id = (int)sh.sid[16 * g + col] - 4 * comp;
#pragma unroll
                for (int m = 0; m < M; ++m) {
                    const f32x4 d = __builtin_amdgcn_mfma_f32_16x16x4f32(A[m], b, f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        part[m][r] = fmaf(id == 16 * m + r ? 0.f : w, __builtin_amdgcn_exp2f(d[r]), part[m][r]);
                }
            }
        } else {
#pragma unroll(M < 3 ? 2 : 1)
            for (int g = 0; g < n16; ++g) {
                const float b = B[64 * g], w = sh.sw[16 * g + col];
#pragma unroll
                for (int m = 0; m < M; ++m) {
                    const f32x4 d = __builtin_amdgcn_mfma_f32_16x16x4f32(A[m], b, f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
#pragma unroll
                    for (int r = 0; r < 4; ++r) part[m][r] = fmaf(w, __builtin_amdgcn_exp2f(d[r]), part[m][r]);
                }
            }
        }
        if (!flush) return;
        // at most 32 terms a value; the 16 source columns, halving the columns and the
        // values together, then the other columns
#pragma unroll
        for (int m = 0; m < M; ++m) {
            const bool hi2 = (lane & 2) != 0, hi1 = (lane & 1) != 0;
            const float a = (hi2 ? part[m][2] : part[m][0]) + dpp<0x4e>(hi2 ? part[m][0] : part[m][2]);   // lane ^ 2
            const float b = (hi2 ? part[m][3] : part[m][1]) + dpp<0x4e>(hi2 ? part[m][1] : part[m][3]);
            float v = (hi1 ? b : a) + dpp<0xb1>(hi1 ? a : b);   // lane ^ 1
            v += dpp<0x124>(v);                                 // row_ror 4, 8
            v += dpp<0x128>(v);
            total[m] += (double)v;
#pragma unroll
            for (int r = 0; r < 4; ++r) part[m][r] = 0.f;
        }
    };
    p2p_sources<NW>(L, lst, len, tf, nt, wave, sh, stage, use);
    // target 16 m + 4 c + q from lane 16 c + q to lane 16 m + 4 c + q
    double s = 0.0;
#pragma unroll
    for (int m = 0; m < M; ++m) {
        const double to = __shfl(total[m], ((lane & 12) << 2) | (lane & 3), 64);
        if (comp == m) s = to;
    }
    return s;
}

// Wave `wave` of the NW that share the target leaf of task t (the same for all of them);
// red: one row of 64 per wave (NW > 1).
template <int NW>
__device__ inline void p2p_leaf(const LeafSet &L, const LeafTask &t, int wave, P2PShared &sh, double (*red)[64]) {
    const int lane = threadIdx.x & 63, len = t.len;
    const int32_t tf = t.first, tn = t.count, *lst = t.lst;
    const float *ct = t.ct;
    const bool matrix = __builtin_amdgcn_readfirstlane((int)(1.7320508f * t.half * L.k_scale <= kMatrixReach));
    sh.sp[kP2PChunk + lane] = make_float4(0.f, 0.f, 0.f, 0.f);
    sh.sid[kP2PChunk + lane] = kNoTarget;
    for (int t0 = 0; t0 < tn; t0 += 64) {
        const int nt = __builtin_amdgcn_readfirstlane(tn - t0 < 64 ? tn - t0 : 64);
        double s = 0.0;
#define MSP_P2P(F, K) F<NW, K>(L, lst, len, ct, tf + t0, nt, wave, sh)
        bool again = false;
        if (matrix) {
            if (nt <= 16) s = MSP_P2P(p2p_block_matrix, 1);
            else if (nt <= 32) s = MSP_P2P(p2p_block_matrix, 2);
            else if (nt <= 48) s = MSP_P2P(p2p_block_matrix, 3);
            else s = MSP_P2P(p2p_block_matrix, 4);
            // w exp2(t^2 - d^2) of weights beyond 2^127 / 2 leaves float32 where w exp2(-d^2) does
            // not: these by differences
            again = __ballot(lane < nt && !(fabs(s) <= 3.4028234663852886e38)) != 0;
        }
        if (!matrix || again) {
            if (nt <= 9) s = MSP_P2P(p2p_block_vector, 1);
            else if (nt <= 18) s = MSP_P2P(p2p_block_vector, 2);
            else s = MSP_P2P(p2p_block_vector, 4);
            if (again && lane < nt) s /= target_factor(L, tf + t0 + lane, ct);
        }
#undef MSP_P2P
        if constexpr (NW > 1) {
            // the waves in order
            red[wave][lane] = s;
            __syncthreads();
            if (wave == 0 && lane < nt) {
                s = 0.0;
#pragma unroll
                for (int q = 0; q < NW; ++q) s += red[q][lane];
            }
        }
        if (wave == 0 && lane < nt) {
            const int32_t ti = tf + t0 + lane;
            if (matrix) s *= target_factor(L, ti, ct);
            L.usort[ti] = ld_global(L.tflag, ti) ? (float)s : 0.f;
        }
        if constexpr (NW > 1) __syncthreads();   // red is free again
    }
}

}  // namespace
}  // namespace msp
