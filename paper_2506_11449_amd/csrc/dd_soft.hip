// Soft TopK weights of the candidate diagonals and the scaling of the active diagonals by them
// (Sec. 3.2, Eq. 4 and Eq. 5), forward and backward.  O(D) and O(K*L) element-wise work with block
// reductions: launch-bound, one workgroup per score vector / per diagonal, fixed reduction order.
#include "dd_common.h"
#include "dd_launch.h"
#include "dd_select_block.h"
#include "dd_soft_block.h"

namespace dd {

constexpr int kScaleThreads = 256;  // kernels that run over the K x L values

// SLOTS: candidates that a thread holds in registers, 0 (1024 threads): read from memory by each pass
template <int THREADS, int SLOTS>
__global__ __launch_bounds__(THREADS) void soft_topk_kernel(int D, float k_over_1, float inv_temp,
                                                            const float *__restrict__ scores,
                                                            float *__restrict__ alpha_tilde)
{
    const float *row = scores + size_t(blockIdx.x) * D;
    float *out = alpha_tilde + size_t(blockIdx.x) * D;
    if constexpr (SLOTS > 0) {
        float a[SLOTS];
        hold<THREADS, SLOTS>(D, row, a);
        soft_topk_held<THREADS, SLOTS>(D, k_over_1, inv_temp, a, out);
    } else {
        soft_topk_block(D, k_over_1, inv_temp, row, out);
    }
}

// d a_i = (K / temp) * s_i * (m_i g_i - sum_j m_j g_j s_j),  m_j = [K s_j < 1]
template <int THREADS, int SLOTS>
__global__ __launch_bounds__(THREADS) void soft_topk_bwd_kernel(int D, float k_over_1, float inv_temp,
                                                                const float *__restrict__ scores,
                                                                const float *__restrict__ g,
                                                                float *__restrict__ dscores)
{
    const float *a = scores + size_t(blockIdx.x) * D, *gb = g + size_t(blockIdx.x) * D;
    float *out = dscores + size_t(blockIdx.x) * D;
    if constexpr (SLOTS > 0) {
        __shared__ HeldScratch held;
        float x[SLOTS], g_held[SLOTS], s[SLOTS], part[SLOTS];
        hold<THREADS, SLOTS>(D, a, x);
        hold<THREADS, SLOTS>(D, gb, g_held);
        const float inv_s = 1.f / exponentials_held<THREADS, SLOTS>(D, inv_temp, x, held, s);
#pragma unroll
        for (int j = 0; j < SLOTS; ++j) {
            s[j] *= inv_s;
            if (!(k_over_1 * s[j] < 1.f)) g_held[j] = 0.f;
            part[j] = j * THREADS + int(threadIdx.x) < D && k_over_1 * s[j] < 1.f ? g_held[j] * s[j] : 0.f;
        }
        const float dot = sum_held<THREADS, SLOTS>(part, held.waves[2], held.parts[1]);
#pragma unroll
        for (int j = 0; j < SLOTS; ++j)
            if (j * THREADS + int(threadIdx.x) < D) out[j * THREADS + threadIdx.x] = k_over_1 * inv_temp * s[j] * (g_held[j] - dot);
    } else {
        __shared__ SoftScratch scratch;
        const float m = reduce_scores<true>(D, scratch, [&](int i) { return a[i]; });
        const float s = reduce_scores<false>(D, scratch, [&](int i) { return expf((a[i] - m) * inv_temp); });
        const float inv_s = 1.f / s;
        const float dot = reduce_scores<false>(D, scratch, [&](int i) {
            const float si = expf((a[i] - m) * inv_temp) * inv_s;
            return k_over_1 * si < 1.f ? gb[i] * si : 0.f;
        });
        for (int i = threadIdx.x; i < D; i += THREADS) {
            const float si = expf((a[i] - m) * inv_temp) * inv_s;
            const float mg = k_over_1 * si < 1.f ? gb[i] : 0.f;
            out[i] = k_over_1 * inv_temp * si * (mg - dot);
        }
    }
}

// values_eff[k][p] = alpha_tilde[o_k] * V[k][p]
template <class S>
__global__ __launch_bounds__(kScaleThreads) void scale_values_kernel(int L, int D, const int *__restrict__ offsets,
                                                                    const float *__restrict__ alpha_tilde,
                                                                    const typename S::storage *__restrict__ V,
                                                                    typename S::storage *__restrict__ out)
{
    const int k = blockIdx.y, p = blockIdx.x * kScaleThreads + threadIdx.x;
    if (p >= L) return;
    const float a = alpha_tilde[canonical_offset(offsets[k], D)];
    S::store(out + size_t(k) * L + p, a * S::load(V + size_t(k) * L + p));
}

// dV[k][p] = alpha_tilde[o_k] * dValues[k][p];  dots[k] = <dValues[k], V[k]>
template <class S>
__global__ __launch_bounds__(kScaleThreads) void scale_values_bwd_kernel(int L, int D, const int *__restrict__ offsets,
                                                                        const float *__restrict__ alpha_tilde,
                                                                        const typename S::storage *__restrict__ V,
                                                                        const float *__restrict__ dValues,
                                                                        float *__restrict__ dV,
                                                                        float *__restrict__ dots)
{
    __shared__ float scratch[kScaleThreads / 64];
    const int k = blockIdx.x;
    const float a = alpha_tilde[canonical_offset(offsets[k], D)];
    float dot = 0.f;
    for (int p = threadIdx.x; p < L; p += kScaleThreads) {
        const float g = dValues[size_t(k) * L + p];
        dV[size_t(k) * L + p] = a * g;
        dot = fmaf(g, S::load(V + size_t(k) * L + p), dot);
    }
    dot = block_reduce<false, kScaleThreads>(dot, scratch);
    if (threadIdx.x == 0) dots[k] = dot;
}

// dalpha_tilde[i] = sum over the diagonals k with offset i, in index order, of dots[k]
__global__ __launch_bounds__(kScaleThreads) void scatter_alpha_grad_kernel(int D, int K, const int *__restrict__ offsets,
                                                                          const float *__restrict__ dots,
                                                                          float *__restrict__ dalpha)
{
    const int i = blockIdx.x * kScaleThreads + threadIdx.x;
    if (i >= D) return;
    float acc = 0.f;
    for (int k = 0; k < K; ++k)
        if (canonical_offset(offsets[k], D) == i) acc += dots[k];
    dalpha[i] = acc;
}

// the instance for that many threads and candidates per thread
#define DD_SOFT_BY_SLOTS(kernel_, threads_, slots_)                                                     \
    ((threads_) == kSelectThreadsFew ? ((slots_) <= 1    ? kernel_<kSelectThreadsFew, 1>                \
                                        : (slots_) <= 4  ? kernel_<kSelectThreadsFew, 4>                \
                                        : (slots_) <= 8  ? kernel_<kSelectThreadsFew, 8>                \
                                                         : kernel_<kSelectThreadsFew, 16>)              \
                                     : ((slots_) <= 4  ? kernel_<kSelectThreads, 4>                   \
                                        : (slots_) <= 6  ? kernel_<kSelectThreads, 6>                   \
                                        : (slots_) <= 8  ? kernel_<kSelectThreads, 8>                   \
                                        : (slots_) <= 12 ? kernel_<kSelectThreads, 12>                  \
                                        : (slots_) <= 16 ? kernel_<kSelectThreads, 16>                  \
                                                         : kernel_<kSelectThreads, 0>))

hipError_t launch_soft_topk(int batch, int D, int K, float temperature, const float *scores, float *alpha_tilde,
                            hipStream_t stream)
{
    const int threads = select_threads(batch, D);
    hipLaunchKernelGGL(DD_SOFT_BY_SLOTS(soft_topk_kernel, threads, (D + threads - 1) / threads),
                       dim3(batch), dim3(threads), 0, stream, D, float(K), 1.f / temperature, scores, alpha_tilde);
    return hipGetLastError();
}

hipError_t launch_soft_topk_bwd(int batch, int D, int K, float temperature, const float *scores, const float *g,
                                float *dscores, hipStream_t stream)
{
    const int threads = select_threads(batch, D);
    hipLaunchKernelGGL(DD_SOFT_BY_SLOTS(soft_topk_bwd_kernel, threads, (D + threads - 1) / threads),
                       dim3(batch), dim3(threads), 0, stream, D, float(K), 1.f / temperature, scores, g, dscores);
    return hipGetLastError();
}

hipError_t launch_scale_values(int K, int L, int D, bool bf16, const int *offsets, const float *alpha_tilde,
                               const void *V, void *out, hipStream_t stream)
{
    dim3 grid((L + kScaleThreads - 1) / kScaleThreads, K);
    if (bf16)
        hipLaunchKernelGGL(scale_values_kernel<BF16>, grid, dim3(kScaleThreads), 0, stream, L, D, offsets, alpha_tilde,
                           static_cast<const uint16_t *>(V), static_cast<uint16_t *>(out));
    else
        hipLaunchKernelGGL(scale_values_kernel<F32>, grid, dim3(kScaleThreads), 0, stream, L, D, offsets, alpha_tilde,
                           static_cast<const float *>(V), static_cast<float *>(out));
    return hipGetLastError();
}

hipError_t launch_scale_values_bwd(int K, int L, int D, bool bf16, const int *offsets, const float *alpha_tilde,
                                   const void *V, const float *dValues, float *dV, float *dalpha, float *dots,
                                   hipStream_t stream)
{
    if (bf16)
        hipLaunchKernelGGL(scale_values_bwd_kernel<BF16>, dim3(K), dim3(kScaleThreads), 0, stream, L, D, offsets,
                           alpha_tilde, static_cast<const uint16_t *>(V), dValues, dV, dots);
    else
        hipLaunchKernelGGL(scale_values_bwd_kernel<F32>, dim3(K), dim3(kScaleThreads), 0, stream, L, D, offsets,
                           alpha_tilde, static_cast<const float *>(V), dValues, dV, dots);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(scatter_alpha_grad_kernel, dim3((D + kScaleThreads - 1) / kScaleThreads), dim3(kScaleThreads), 0,
                       stream, D, K, offsets, dots, dalpha);
    return hipGetLastError();
}

}  // namespace dd
