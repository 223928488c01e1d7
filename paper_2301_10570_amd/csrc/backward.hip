// Derivatives of L = sum_i g_i u(t_i) (targets i) with respect to the weights, the
// positions and sigma.  With K = exp(-|t - s|^2 / sigma^2):
//   dL/dw_j     = v(s_j),  v(x) = sum_i g_i K(t_i, x)          (the transposed sum)
//   dL/dx_k     = g_k grad u(x_k) + w_k grad v(x_k)             (a point may be both)
//   dL/dsigma   = sum_i g_i [ (sigma/2) lap u(t_i) + (3/sigma) u(t_i) ]
// using dK/dsigma = (sigma/2) lap_t K + (3/sigma) K (the heat equation of the
// Gaussian).  Two field evaluations give everything: u with gradient and
// Laplacian (weights w), and v with gradient (weights g at the targets), both by
// the expansion route (L2P with derivatives) or the direct route (P2P with
// derivatives).
#include "grad_common.hpp"

#include <cmath>

namespace msp {
namespace {

constexpr int kBlock = 256;

__global__ void k_target_weights(const float *g, const uint8_t *is_target, int64_t n, float *gt) {
    int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    gt[i] = (!is_target || is_target[i]) ? g[i] : 0.f;
}

// Both fields' weights into key order: w into the records, the target weights into g2.
__global__ void k_stage_both(const float *w, const float *gt, const int32_t *perm, int64_t n, float4 *ps, float *g2) {
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int32_t j = perm[i];
    ps[i].w = w[j];
    g2[i] = gt[j];
}

// P2P with derivatives, NW wavefronts per target leaf.
template <int NW, bool TWO>
__global__ void __launch_bounds__(NW * 64, NW > 1 ? 4 : 6)
k_p2p_grad(GradLeafSet L, const float *g2, int stride, int want_lap) {
    __shared__ GradShared sh[NW];
    __shared__ GradBlock own;
    GradBlock &bk = NW > 1 ? own : *reinterpret_cast<GradBlock *>(sh[0].src);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const LeafTask t = uniform_copy(leaf_task(L, (int64_t)blockIdx.x, 0));
    if (t.count > 0) p2p_grad_leaf<NW, TWO>(L, g2, t, stride, want_lap, wave, sh[wave], bk);
}

// Eight wavefronts per leaf while the tree has fewer leaves than the chip has wavefront
// slots, one beyond.
template <bool TWO>
void launch_p2p_grad(const GradLeafSet &L, const float *g2, int stride, int want_lap, hipStream_t s) {
    const dim3 grid((unsigned)L.n_nodes);
    if (p2p_waves(L.n_nodes) > 1)
        hipLaunchKernelGGL(HIP_KERNEL_NAME(k_p2p_grad<8, TWO>), grid, dim3(512), 0, s, L, g2, stride, want_lap);
    else
        hipLaunchKernelGGL(HIP_KERNEL_NAME(k_p2p_grad<1, TWO>), grid, dim3(64), 0, s, L, g2, stride, want_lap);
}

// Per point of the input order j: the key-order record of its point (64 bytes,
// one aligned segment: A value, gradient, Laplacian, then B value, gradient)
// combined into the gradients; per-block partial sums of the sigma derivative.
__global__ void k_combine(int64_t n, const int32_t *iperm, const float *gt, const float *w,
                          const float *rec, int want_w, int want_pos, int want_sigma, double sigma,
                          int exclude_self, float *grad_w, float *grad_x, float *grad_y, float *grad_z,
                          double *partial) {
    __shared__ double red[kBlock];
    const int64_t j = blockIdx.x * (int64_t)kBlock + threadIdx.x;
    double ds = 0.0;
    if (j < n)
        ds = combine_point(reinterpret_cast<const float4 *>(rec + (int64_t)iperm[j] * kRec), gt[j],
                           want_pos ? w[j] : 0.f, want_w, want_pos, want_sigma, sigma, exclude_self,
                           want_w ? grad_w + j : nullptr, want_pos ? grad_x + j : nullptr,
                           want_pos ? grad_y + j : nullptr, want_pos ? grad_z + j : nullptr);
    red[threadIdx.x] = ds;
    __syncthreads();
    for (int st = kBlock / 2; st > 0; st >>= 1) {
        if ((int)threadIdx.x < st) red[threadIdx.x] += red[threadIdx.x + st];
        __syncthreads();
    }
    if (threadIdx.x == 0 && partial) partial[blockIdx.x] = red[0];
}

__global__ void k_sum_partials(const double *partial, int64_t m, double *out) {
    __shared__ double red[kBlock];
    double s = 0.0;
    for (int64_t k = threadIdx.x; k < m; k += kBlock) s += partial[k];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int st = kBlock / 2; st > 0; st >>= 1) {
        if ((int)threadIdx.x < st) red[threadIdx.x] += red[threadIdx.x + st];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[0] = red[0];
}

}  // namespace

// Value, gradient and Laplacian of the field of the staged weights ps.w (and, with
// g2, value and gradient of the field of the weights g2, at out + 5) by the direct
// route, whose lists the handle holds.
static int direct_field_grad(msp_tree *t, const msp_fgt_params *prm, const float *g2, float *out, int stride,
                             int want_lap, hipStream_t s) {
    const double sig = prm->sigma;
    const GradLeafSet L{t->n_nodes, t->nfirst.as<int32_t>(), t->ncount.as<int32_t>(), t->nnchild.as<int32_t>(),
                        t->nlevel.as<int32_t>(), t->nix.as<int32_t>(), t->niy.as<int32_t>(), t->niz.as<int32_t>(),
                        BoxGeo{{t->geo.lo[0], t->geo.lo[1], t->geo.lo[2]}, t->geo.side},
                        LeafLists{t->list_off.as<int64_t>(), t->list_stride, t->list_cnt.as<int32_t>(),
                                  t->list_idx.as<int32_t>()},
                        t->ps.as<float4>(), (float)(-1.4426950408889634 / (sig * sig)), (float)(1.0 / (sig * sig)),
                        out};
    PhaseScope ps(&t->timing, PH_P2P, s);
    if (g2) launch_p2p_grad<true>(L, g2, stride, want_lap, s);
    else launch_p2p_grad<false>(L, nullptr, stride, want_lap, s);
    MSP_CHECK_LAUNCH();
    return MSP_OK;
}

int fgt_backward(msp_tree *t, const float *w, const uint8_t *is_target, const msp_fgt_params *prm,
                 const float *grad_u, float *grad_w, float *grad_x, float *grad_y, float *grad_z,
                 double *grad_sigma, hipStream_t s) {
    const int64_t n = t->n;
    FgtPlan pl;
    MSP_TRY(plan_fgt(t, prm, &pl));
    const int64_t nb = n > 0 ? n : 1;
    const int64_t nblk = (nb + kBlock - 1) / kBlock;
    // scratch: one 64-byte record per point in key order (A: value, gradient,
    // Laplacian; B: value, gradient), gt in input order and in key order, block partials
    MSP_TRY(t->bwd.ensure((size_t)nb * (kRec + 2) * 4 + (size_t)nblk * 8 + 64));
    float *rec = t->bwd.as<float>();
    float *gt = rec + (size_t)nb * kRec;
    float *g2 = gt + nb;
    double *partial = reinterpret_cast<double *>(g2 + nb);
    if (n == 0) {
        // a kernel rather than a memset, so that the sequence can be captured into a graph
        if (grad_sigma) {
            hipLaunchKernelGGL(k_sum_partials, dim3(1), dim3(kBlock), 0, s, partial, (int64_t)0, grad_sigma);
            MSP_CHECK_LAUNCH();
        }
        return MSP_OK;
    }
    const bool needA = grad_x || grad_sigma;
    const bool needB = grad_w || grad_x;
    MSP_TRY(ensure_iperm(t, s));
    hipLaunchKernelGGL(k_target_weights, dim3(grid_for(n, kBlock)), dim3(kBlock), 0, s, grad_u, is_target,
                       n, gt);
    MSP_CHECK_LAUNCH();
    if (pl.route == MSP_ROUTE_FGT) {
        if (needA) MSP_TRY(fgt_field_grad(t, pl, prm, w, rec, kRec, grad_sigma ? 1 : 0, s));
        if (needB) MSP_TRY(fgt_field_grad(t, pl, prm, gt, rec + 5, kRec, 0, s));
    } else {
        msp_fgt_params q = *prm;
        q.flags &= ~(uint32_t)MSP_EXCLUDE_SELF;
        MSP_TRY(direct_route_lists(t, &q, s));
        if (needA && needB) {   // both fields in one pass: one exponential per pair serves both
            ++t->ps_gen;
            hipLaunchKernelGGL(k_stage_both, dim3(grid_for(n, kBlock)), dim3(kBlock), 0, s, w, gt,
                               t->perm.as<int32_t>(), n, t->ps.as<float4>(), g2);
            MSP_CHECK_LAUNCH();
            MSP_TRY(direct_field_grad(t, &q, g2, rec, kRec, grad_sigma ? 1 : 0, s));
        } else if (needA || needB) {
            MSP_TRY(stage_inputs(t, needA ? w : gt, nullptr, s));
            MSP_TRY(direct_field_grad(t, &q, nullptr, needA ? rec : rec + 5, kRec, needA && grad_sigma ? 1 : 0, s));
        }
    }
    {
        PhaseScope ps(&t->timing, PH_BACKWARD, s);
        hipLaunchKernelGGL(k_combine, dim3((unsigned)nblk), dim3(kBlock), 0, s, n, t->iperm.as<int32_t>(), gt,
                           w, rec, grad_w && needB ? 1 : 0, grad_x ? 1 : 0, grad_sigma ? 1 : 0,
                           (double)prm->sigma, (prm->flags & MSP_EXCLUDE_SELF) ? 1 : 0, grad_w, grad_x,
                           grad_y, grad_z, partial);
        MSP_CHECK_LAUNCH();
        if (grad_sigma) {
            hipLaunchKernelGGL(k_sum_partials, dim3(1), dim3(kBlock), 0, s, partial, nblk, grad_sigma);
            MSP_CHECK_LAUNCH();
        }
    }
    return MSP_OK;
}

}  // namespace msp
