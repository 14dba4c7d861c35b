// Hard TopK re-selection of active diagonals (Sec. 3.2, Eq. 4): which K of the D importance
// scores are kept.  One workgroup per score vector, integer comparisons only, so the result
// is the same on every run and on every device.
// The method itself is in dd_select_block.h.
#include "dd_common.h"
#include "dd_launch.h"
#include "dd_select_block.h"
#include "dd_soft_block.h"

namespace dd {

template <int THREADS, int SLOTS>
__global__ __launch_bounds__(THREADS) void select_topk_kernel(int D, int K, const float *__restrict__ scores,
                                                              int *__restrict__ out)
{
    __shared__ __attribute__((aligned(16))) SelectScratch<THREADS, SLOTS> scratch;
    select_topk_block<THREADS, SLOTS>(D, K, scores + size_t(blockIdx.x) * D, scratch, out + size_t(blockIdx.x) * K);
}

// The selection and, in the same launch, the soft TopK weights of the same scores (Eq. 4 picks the diagonals, Eq. 5
// weighs them): the workgroup that has just ranked a score vector also normalises it.
template <int THREADS, int SLOTS>
__global__ __launch_bounds__(THREADS) void select_soft_kernel(int D, int K, float inv_temp,
                                                              const float *__restrict__ scores, int *__restrict__ out,
                                                              float *__restrict__ alpha_tilde)
{
    __shared__ __attribute__((aligned(16))) SelectScratch<THREADS, SLOTS> scratch;
    const float *row = scores + size_t(blockIdx.x) * D;
    int *chosen = out + size_t(blockIdx.x) * K;
    float *weights = alpha_tilde + size_t(blockIdx.x) * D;
    if constexpr (SLOTS <= kSoftHeldSlots) {
        float a[SLOTS];
        hold<THREADS, SLOTS>(D, row, a);
        select_held_block<THREADS, SLOTS>(D, K, a, scratch, chosen);
        soft_topk_held<THREADS, SLOTS>(D, float(K), inv_temp, a, weights);
    } else {
        select_topk_block<THREADS, SLOTS>(D, K, row, scratch, chosen);
        soft_topk_block(D, float(K), inv_temp, row, weights);
    }
}

// the instance for that many threads and candidates per thread, by the name of a template of the two
#define DD_BY_SLOTS(kernel_, threads_, slots_)                                                          \
    ((threads_) == kSelectThreadsFew ? ((slots_) <= 1   ? kernel_<kSelectThreadsFew, 1>                 \
                                        : (slots_) <= 2 ? kernel_<kSelectThreadsFew, 2>                 \
                                        : (slots_) <= 3 ? kernel_<kSelectThreadsFew, 3>                 \
                                        : (slots_) <= 4 ? kernel_<kSelectThreadsFew, 4>                 \
                                        : (slots_) <= 6 ? kernel_<kSelectThreadsFew, 6>                 \
                                        : (slots_) <= 8 ? kernel_<kSelectThreadsFew, 8>                 \
                                                        : kernel_<kSelectThreadsFew, 16>)               \
                                     : ((slots_) <= 3  ? kernel_<kSelectThreads, 3>                   \
                                        : (slots_) <= 4  ? kernel_<kSelectThreads, 4>                   \
                                        : (slots_) <= 8  ? kernel_<kSelectThreads, 8>                   \
                                        : (slots_) <= 16 ? kernel_<kSelectThreads, 16>                  \
                                                         : kernel_<kSelectThreads, kSelectMaxSlots>))

hipError_t launch_select_soft(int batch, int D, int K, float temperature, const float *scores, int *out,
                              float *alpha_tilde, hipStream_t stream)
{
    const int threads = select_threads(batch, D), slots = (D + threads - 1) / threads;
    hipLaunchKernelGGL(DD_BY_SLOTS(select_soft_kernel, threads, slots), dim3(batch), dim3(threads), 0, stream, D, K,
                       1.f / temperature, scores, out, alpha_tilde);
    return hipGetLastError();
}

hipError_t launch_select(int batch, int D, int K, const float *scores, int *out, hipStream_t stream)
{
    if (batch > 256 && D <= 256) {  // many short vectors: fewer waves yet (4000 x 64 scores 5.2 us, with 256 threads 7.8)
        hipLaunchKernelGGL((D <= 128 ? select_topk_kernel<128, 1> : select_topk_kernel<128, 2>), dim3(batch), dim3(128), 0, stream,
                           D, K, scores, out);
        return hipGetLastError();
    }
    const int threads = select_threads(batch, D), slots = (D + threads - 1) / threads;
    hipLaunchKernelGGL(DD_BY_SLOTS(select_topk_kernel, threads, slots), dim3(batch), dim3(threads), 0, stream, D, K, scores, out);
    return hipGetLastError();
}
#undef DD_BY_SLOTS

}  // namespace dd
