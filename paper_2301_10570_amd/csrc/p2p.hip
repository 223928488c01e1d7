// Direct evaluation of the Gaussian sum (Eq. (8)).
//
// Near-field route: for every leaf of the octree, the list of source leaves whose
// boxes come within the cutoff radius of its box (interaction lists built by walks
// of the node table), then P2P: one to sixteen wavefronts per target leaf, source
// leaves staged through LDS.
//
// All-pairs baseline: every target against every source with no tree and no
// cutoff, sources streamed through LDS in tiles.
//
// exp(-d^2/sigma^2) is evaluated as exp2(-(k d)^2) with k^2 = log2(e)/sigma^2.
#include "internal.hpp"
#include "p2p_leaf.hpp"

#include <cmath>

namespace msp {
namespace {

constexpr int kBlock = 256;
// trees of at most this many nodes keep their lists as one row of n_nodes entries per
// node (16 MB at most): the rows need no count before they are filled, so no
// second walk, no prefix sum and no host wait for their total
constexpr int64_t kRowNodes = 2048;
// pending nodes of one wavefront's walk, and what a walk that takes one node at a time
// can add to them (7 per level and the last one's children)
constexpr int kWalkCap = 1024, kWalkTail = 8 * (kDepth + 1);

// The source leaves within reach of each leaf, in key order, one wavefront per node
// (inner nodes have empty lists).  A walk in key order over a stack in LDS whose top is
// the first node to come: a step takes up to 64 nodes from the top, one per lane (fewer
// when the stack is nearly full: a step adds at most 7 per node it takes), drops those
// out of reach, writes the leaves that come before the first inner node and puts the
// rest back, inner nodes as their children, leaves within reach marked as such (~u).
// One thread per leaf walking alone waited for six dependent loads per node: 395 us for
// each of the two walks (count, fill) over 5,003 points; this one takes 12 us.
// cnt == NULL: the counts are there already; lst == NULL: count only.
__global__ void __launch_bounds__(kBlock) k_lists(int64_t n_nodes, const int32_t *nlevel, const int32_t *nix,
                                                  const int32_t *niy, const int32_t *niz,
                                                  const int32_t *nfchild, const int32_t *nnchild, BoxGeo geo,
                                                  float r2, int unlimited, const int64_t *off, int64_t stride,
                                                  int32_t *cnt, int32_t *lst) {
    __shared__ int32_t stacks[kBlock / 64][kWalkCap];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t v = blockIdx.x * (int64_t)(kBlock / 64) + wave;
    if (v >= n_nodes) return;
    if (nnchild[v] != 0) {
        if (cnt && lane == 0) cnt[v] = 0;
        return;
    }
    int32_t *stk = stacks[wave];
    float ct[3], ht;
    node_box(geo, nlevel[v], nix[v], niy[v], niz[v], ct, ht);
    int32_t *row = lst ? lst + (stride > 0 ? v * stride : off[v]) : nullptr;
    if (lane == 0) stk[0] = 0;
    int sp = 1;
    int32_t c = 0;
    while (sp > 0) {
        const int room = (kWalkCap - kWalkTail - sp) / 7;
        int take = sp < 64 ? sp : 64;
        take = take < room ? take : (room > 1 ? room : 1);
        sp -= take;
        wave_sync();
        const int32_t e = lane < take ? stk[sp + take - 1 - lane] : 0;
        wave_sync();   // the popped slots may be written again
        bool leaf = lane < take && e < 0, inner = false;
        const int32_t u = e < 0 ? ~e : e;
        int nc = 0;
        int32_t f = 0;
        if (lane < take && e >= 0) {
            nc = nnchild[u];
            f = nfchild[u];
            float cs[3], hs;
            node_box(geo, nlevel[u], nix[u], niy[u], niz[u], cs, hs);
            float d2 = 0.f;
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                const float gap = fmaxf(fabsf(ct[a] - cs[a]) - (ht + hs), 0.f);
                d2 = fmaf(gap, gap, d2);
            }
            const bool in = unlimited || !(d2 > r2);
            leaf = in && nc == 0;
            // children sit one level deeper, so the walk ends within max_depth levels; the
            // bounds only protect against a corrupt table
            inner = in && nc > 0 && nc <= 8 && f > u && f + nc <= n_nodes;
        }
        const unsigned long long leaves = __ballot(leaf), inners = __ballot(inner);
        // the leaves before the first inner node are next in key order
        const unsigned long long ready = inners ? leaves & ((inners & (0 - inners)) - 1) : leaves;
        const bool mine = (ready >> lane) & 1;
        if (row && mine) row[c + __popcll(ready & ((1ull << lane) - 1))] = u;
        c += __popcll(ready);
        const int k = inner ? nc : (leaf && !mine ? 1 : 0);
        const int incl = p2p_incl_scan(k);
        const int all = __builtin_amdgcn_readfirstlane(__shfl(incl, 63, 64));
        if (sp + all > kWalkCap) continue;
        const int top = sp + all - 1 - (incl - k);
        if (inner)
            for (int q = 0; q < nc; ++q) stk[top - q] = f + q;
        else if (k)
            stk[top] = ~u;
        sp += all;
    }
    if (cnt && lane == 0) cnt[v] = c;
}

// Exclusive prefix sum of cnt into off, the total into off[n]: one block, 1024
// coalesced entries per round.
__global__ void __launch_bounds__(1024) k_scan_i32_to_i64(const int32_t *cnt, int64_t n, int64_t *off) {
    __shared__ int64_t part[16];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int64_t run = 0;
    for (int64_t b0 = 0; b0 < n; b0 += 1024) {
        const int64_t i = b0 + threadIdx.x;
        const int64_t x = i < n ? cnt[i] : 0;
        int64_t v = x;
        for (int o = 1; o < 64; o <<= 1) {
            const int64_t t = __shfl_up(v, o, 64);
            if (lane >= o) v += t;
        }
        if (lane == 63) part[wave] = v;
        __syncthreads();
        int64_t before = run, all = 0;
        for (int q = 0; q < 16; ++q) {
            if (q < wave) before += part[q];
            all += part[q];
        }
        if (i < n) off[i] = before + v - x;
        run += all;
        __syncthreads();
    }
    if (threadIdx.x == 0) off[n] = run;
}

// NW wavefronts per target leaf (non-leaf nodes return at once): a block per node, or
// for NW = 1 four nodes per block, held to 80 registers: with short lists the pass waits for
// loads (150,000 points in leaves of up to 8, lists of 30: 90 us with 112 registers, 75 us).
template <int NW>
__global__ void __launch_bounds__(NW == 1 ? 256 : NW * 64, NW == 1 ? 6 : 4) k_p2p(LeafSet ls) {
    constexpr int W = NW == 1 ? 4 : NW;
    __shared__ P2PShared sh[W];
    __shared__ double red[NW > 1 ? NW : 1][64];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const LeafTask t = uniform_copy(leaf_task(ls, NW == 1 ? (int64_t)blockIdx.x * 4 + wave : (int64_t)blockIdx.x, 0));
    if (t.count > 0) p2p_leaf<NW>(ls, t, NW == 1 ? 0 : wave, sh[wave], red);
}

// All-pairs baseline.  A block of sixteen wavefronts takes T targets; a wavefront's
// lanes split into 64 / T groups, and the sources go round the wavefronts in chunks of
// 128, staged in LDS by the wavefront that uses them (no block barrier until the end).
// Bound by the vector units (ten issues and one exponential per pair).  With one target
// per thread and every source in each block, 16,384 targets made 64 blocks on 256
// compute units: 7.38 ms against 262,144 sources (5.8e11 pairs/s).
constexpr int kDirWaves = 16, kDirChunk = 128;
template <int T>
__global__ void __launch_bounds__(kDirWaves * 64, 8) k_direct(const float *tx, const float *ty, const float *tz,
                                                              int64_t nt, const float *sx, const float *sy,
                                                              const float *sz, const float *w, int64_t ns,
                                                              float neg_c, float *u) {
    constexpr int G = 64 / T;                        // source groups of a wavefront
    constexpr int STEPS = kDirChunk / G;             // sources of a group in a chunk
    constexpr int U = STEPS < 4 ? STEPS : 4;         // independent partial sums
    __shared__ float4 tile[kDirWaves][kDirChunk];
    __shared__ double red[kDirWaves][T];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int grp = lane / T;
    const int64_t i = blockIdx.x * (int64_t)T + lane % T;
    const bool valid = i < nt;
    const float x = valid ? tx[i] : 0.f, y = valid ? ty[i] : 0.f, z = valid ? tz[i] : 0.f;
    double total = 0.0;
    float4 nxt[2];
    // records past the last source have w = 0, so a full chunk can be summed
    auto fetch = [&](int64_t s0) {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int64_t j = s0 + k * 64 + lane;
            nxt[k] = j < ns ? make_float4(sx[j], sy[j], sz[j], w[j]) : make_float4(0.f, 0.f, 0.f, 0.f);
        }
    };
    const int64_t step = (int64_t)kDirWaves * kDirChunk;
    int64_t s0 = (int64_t)wave * kDirChunk;
    if (s0 < ns) fetch(s0);
    for (; s0 < ns; s0 += step) {
        wave_sync();
        tile[wave][lane] = nxt[0];
        tile[wave][64 + lane] = nxt[1];
        wave_sync();
        if (s0 + step < ns) fetch(s0 + step);
        float part[U];
#pragma unroll
        for (int k = 0; k < U; ++k) part[k] = 0.f;
#pragma unroll(STEPS / U < 4 ? STEPS / U : 4)
        for (int it = 0; it < STEPS; it += U) {
#pragma unroll
            for (int k = 0; k < U; ++k) {
                const float4 q = tile[wave][(it + k) * G + grp];
                const float dx = x - q.x, dy = y - q.y, dz = z - q.z;
                part[k] = fmaf(q.w, __builtin_amdgcn_exp2f(fmaf(dx, dx, fmaf(dy, dy, dz * dz)) * neg_c), part[k]);
            }
        }
        float sum = part[0];
        if constexpr (U == 4) sum = (part[0] + part[1]) + (part[2] + part[3]);
        else if constexpr (U == 2) sum = part[0] + part[1];
        total += (double)sum;
    }
    // groups, then wavefronts, in a fixed order
    for (int o = T; o < 64; o <<= 1) total += __shfl_xor(total, o, 64);
    if (lane < T) red[wave][lane] = total;
    __syncthreads();
    if (threadIdx.x < T && valid) {
        double sum = 0.0;
#pragma unroll
        for (int k = 0; k < kDirWaves; ++k) sum += red[k][lane];
        u[i] = (float)sum;
    }
}

}  // namespace

namespace {
int walk_lists(msp_tree *t, const msp_fgt_params *prm, int64_t stride, int32_t *cnt, int32_t *lst, hipStream_t s) {
    const BoxGeo geo{{t->geo.lo[0], t->geo.lo[1], t->geo.lo[2]}, t->geo.side};
    const bool unlimited = !(prm->cutoff_sigmas > 0.f);
    const float R = unlimited ? 0.f : prm->cutoff_sigmas * prm->sigma;
    hipLaunchKernelGGL(k_lists, dim3(grid_for(t->n_nodes, kBlock / 64)), dim3(kBlock), 0, s, t->n_nodes,
                       t->nlevel.as<int32_t>(), t->nix.as<int32_t>(), t->niy.as<int32_t>(), t->niz.as<int32_t>(),
                       t->nfchild.as<int32_t>(), t->nnchild.as<int32_t>(), geo, R * R, unlimited ? 1 : 0,
                       t->list_off.as<int64_t>(), stride, cnt, lst);
    MSP_CHECK_LAUNCH();
    return MSP_OK;
}
}  // namespace

int direct_route_counts(msp_tree *t, const msp_fgt_params *prm, hipStream_t s) {
    const int64_t nn = t->n_nodes;
    if (t->n == 0) return MSP_OK;
    if (t->counts_valid && t->list_sigma == prm->sigma && t->list_cutoff == prm->cutoff_sigmas) return MSP_OK;
    PhaseScope ps(&t->timing, PH_LISTS, s);
    t->lists_valid = false;
    t->counts_valid = false;
    MSP_TRY(t->list_cnt.ensure(nn * 4));
    MSP_TRY(t->list_off.ensure((nn + 1) * 8));
    MSP_TRY(walk_lists(t, prm, 0, t->list_cnt.as<int32_t>(), nullptr, s));
    hipLaunchKernelGGL(k_scan_i32_to_i64, dim3(1), dim3(1024), 0, s, t->list_cnt.as<int32_t>(), nn,
                       t->list_off.as<int64_t>());
    MSP_CHECK_LAUNCH();
    int64_t total = 0;
    MSP_HIP(hipMemcpyAsync(&total, t->list_off.as<int64_t>() + nn, 8, hipMemcpyDeviceToHost, s));
    MSP_HIP(hipStreamSynchronize(s));
    if (total > 0x7fffffffLL)
        return fail(MSP_ENOSPC, "direct route: %lld leaf pairs within the cutoff exceed the list limit",
                    (long long)total);
    t->list_total = total;
    t->list_sigma = prm->sigma;
    t->list_cutoff = prm->cutoff_sigmas;
    t->counts_valid = true;
    return MSP_OK;
}

int direct_route_fill(msp_tree *t, const msp_fgt_params *prm, hipStream_t s) {
    if (t->n == 0) return MSP_OK;
    PhaseScope ps(&t->timing, PH_LISTS, s);
    MSP_TRY(t->list_idx.ensure((t->list_total > 0 ? t->list_total : 1) * 4));
    return walk_lists(t, prm, 0, nullptr, t->list_idx.as<int32_t>(), s);
}

int direct_route_lists(msp_tree *t, const msp_fgt_params *prm, hipStream_t s) {
    if (t->n == 0) return MSP_OK;
    if (t->lists_valid && t->list_sigma == prm->sigma && t->list_cutoff == prm->cutoff_sigmas) return MSP_OK;
    const int64_t nn = t->n_nodes;
    // The lists of a recorded call exist only after a replay: they are not noted as made.
    // Without their lengths (which msp_fgt_forward_query counts) the call is refused.
    const bool recorded = capturing(s);
    if (recorded && !(t->counts_valid && t->list_sigma == prm->sigma && t->list_cutoff == prm->cutoff_sigmas))
        return fail(MSP_EHIP, "the interaction lists of sigma %g are not there and cannot be counted in a call that is "
                    "recorded into a graph", (double)prm->sigma);
    if (nn <= kRowNodes) {
        PhaseScope ps(&t->timing, PH_LISTS, s);
        t->lists_valid = false;
        t->counts_valid = recorded;   // the offsets of compact lists are not written here
        MSP_TRY(t->list_cnt.ensure(nn * 4));
        MSP_TRY(t->list_idx.ensure(nn * nn * 4));
        MSP_TRY(walk_lists(t, prm, nn, t->list_cnt.as<int32_t>(), t->list_idx.as<int32_t>(), s));
        t->list_sigma = prm->sigma;
        t->list_cutoff = prm->cutoff_sigmas;
        t->list_stride = nn;
    } else {
        MSP_TRY(direct_route_counts(t, prm, s));
        MSP_TRY(direct_route_fill(t, prm, s));
        t->list_stride = 0;
    }
    t->lists_valid = !recorded;
    return MSP_OK;
}

int p2p_waves(int64_t n_nodes) {
    // wavefronts per leaf so that a small tree still fills the chip's 8192 wavefront
    // slots; 16 (the largest block) below 1024 nodes.  4,096 points (300 leaves, lists
    // of 45 chunks) took 220 us on one wavefront per leaf and take 24 us on 16.
    int nw = 16;
    while (nw > 1 && n_nodes * nw > 4 * kSharedNodes) nw >>= 1;
    return nw >= 4 ? nw : 1;
}

int direct_route(msp_tree *t, const msp_fgt_params *prm, hipStream_t s, bool lists_ready) {
    const int64_t nn = t->n_nodes;
    if (t->n == 0) return MSP_OK;
    if (!lists_ready) MSP_TRY(direct_route_lists(t, prm, s));
    const LeafSet ls{nn, t->nfirst.as<int32_t>(), t->ncount.as<int32_t>(), t->nnchild.as<int32_t>(),
                     t->nlevel.as<int32_t>(), t->nix.as<int32_t>(), t->niy.as<int32_t>(), t->niz.as<int32_t>(),
                     BoxGeo{{t->geo.lo[0], t->geo.lo[1], t->geo.lo[2]}, t->geo.side},
                     LeafLists{t->list_off.as<int64_t>(), lists_ready ? 0 : t->list_stride,
                               t->list_cnt.as<int32_t>(), t->list_idx.as<int32_t>()},
                     t->ps.as<float4>(), t->tflag.as<uint8_t>(),
                     (float)(std::sqrt(1.4426950408889634) / (double)prm->sigma),
                     (prm->flags & MSP_EXCLUDE_SELF) ? 1 : 0, t->usort.as<float>()};
    PhaseScope ps(&t->timing, PH_P2P, s);
    switch (p2p_waves(nn)) {
        case 16: hipLaunchKernelGGL(k_p2p<16>, dim3((unsigned)nn), dim3(1024), 0, s, ls); break;
        case 8: hipLaunchKernelGGL(k_p2p<8>, dim3((unsigned)nn), dim3(512), 0, s, ls); break;
        case 4: hipLaunchKernelGGL(k_p2p<4>, dim3((unsigned)nn), dim3(256), 0, s, ls); break;
        default: hipLaunchKernelGGL(k_p2p<1>, dim3((unsigned)((nn + 3) / 4)), dim3(256), 0, s, ls);
    }
    MSP_CHECK_LAUNCH();
    return MSP_OK;
}

int direct_all_pairs(const float *tx, const float *ty, const float *tz, int64_t nt, const float *sx,
                     const float *sy, const float *sz, const float *w, int64_t ns, float sigma,
                     float *u, hipStream_t s) {
    if (nt == 0) return MSP_OK;
    const float neg_c = (float)(-1.4426950408889634 / ((double)sigma * sigma));
    // Targets per block.  More of them share a source read from LDS, fewer spread few targets
    // over the chip.  Against 262,144 sources, us with 2, 8, 32, 64 targets per block:
    // 1,024 targets 142, 157, 587, 1,143; 2,048 266, 164, 585, 1,149; 8,192 1,013, 572, 594,
    // 1,142; 12,288 1,508, 844, 1,033, 1,162; 16,384 2,000, 1,114, 1,041, 1,164; 32,768 3,983,
    // 2,203, 1,940, 2,007; 65,536 7,886, 4,365, 3,714, 3,683.  The lines lie where the next
    // size has made one round of two blocks per compute unit (32: 16,384) or wins (8 and
    // 64); the same against 20,000 sources.
#define MSP_DIRECT(T) hipLaunchKernelGGL(k_direct<T>, dim3(grid_for(nt, T)), dim3(kDirWaves * 64), 0, s, tx, ty, \
                                         tz, nt, sx, sy, sz, w, ns, neg_c, u)
    if (nt >= 64 * 1024) MSP_DIRECT(64);
    else if (nt >= 32 * 512) MSP_DIRECT(32);
    else if (nt >= 1280) MSP_DIRECT(8);
    else MSP_DIRECT(2);
#undef MSP_DIRECT
    MSP_CHECK_LAUNCH();
    return MSP_OK;
}

}  // namespace msp
