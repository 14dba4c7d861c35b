// Hard TopK re-selection of active diagonals (Sec. 3.2, Eq. 4): which K of the D importance
// scores are kept.  One workgroup per score vector, integer comparisons only, so the result
// is the same on every run and on every device.
// The method itself is in dd_select_block.h.
#include "dd_common.h"
#include "dd_launch.h"
#include "dd_select_block.h"
#include "dd_soft_block.h"

namespace dd {

template <int SLOTS>
__global__ __launch_bounds__(kSelectThreads) void select_topk_kernel(int D, int K, const float *__restrict__ scores,
                                                                     int *__restrict__ out)
{
    __shared__ __attribute__((aligned(16))) SelectScratch<kSelectThreads, SLOTS> scratch;
    select_topk_block<kSelectThreads, SLOTS>(D, K, scores + size_t(blockIdx.x) * D, scratch, out + size_t(blockIdx.x) * K);
}

// The selection and, in the same launch, the soft TopK weights of the same scores (Eq. 4 picks the diagonals, Eq. 5
// weighs them): the workgroup that has just ranked a score vector also normalises it.
template <int SLOTS>
__global__ __launch_bounds__(kSelectThreads) void select_soft_kernel(int D, int K, float inv_temp,
                                                                     const float *__restrict__ scores,
                                                                     int *__restrict__ out,
                                                                     float *__restrict__ alpha_tilde)
{
    __shared__ __attribute__((aligned(16))) SelectScratch<kSelectThreads, SLOTS> scratch;
    static_assert(kSelectThreads == kSoftThreads, "one workgroup serves both routines");
    select_topk_block<kSelectThreads, SLOTS>(D, K, scores + size_t(blockIdx.x) * D, scratch, out + size_t(blockIdx.x) * K);
    soft_topk_block(D, float(K), inv_temp, scores + size_t(blockIdx.x) * D, alpha_tilde + size_t(blockIdx.x) * D);
}

template <int SLOTS>
static void launch_select_soft_slots(int batch, int D, int K, float temperature, const float *scores, int *out,
                                     float *alpha_tilde, hipStream_t stream)
{
    hipLaunchKernelGGL(select_soft_kernel<SLOTS>, dim3(batch), dim3(kSelectThreads), 0, stream, D, K, 1.f / temperature,
                       scores, out, alpha_tilde);
}

hipError_t launch_select_soft(int batch, int D, int K, float temperature, const float *scores, int *out,
                              float *alpha_tilde, hipStream_t stream)
{
    const int slots = (D + kSelectThreads - 1) / kSelectThreads;
    if (slots <= 1) launch_select_soft_slots<1>(batch, D, K, temperature, scores, out, alpha_tilde, stream);
    else if (slots <= 4) launch_select_soft_slots<4>(batch, D, K, temperature, scores, out, alpha_tilde, stream);
    else if (slots <= 16) launch_select_soft_slots<16>(batch, D, K, temperature, scores, out, alpha_tilde, stream);
    else launch_select_soft_slots<kSelectMaxSlots>(batch, D, K, temperature, scores, out, alpha_tilde, stream);
    return hipGetLastError();
}

hipError_t launch_select(int batch, int D, int K, const float *scores, int *out, hipStream_t stream)
{
    const int slots = (D + kSelectThreads - 1) / kSelectThreads;
    const dim3 grid(batch), block(kSelectThreads);
    if (slots <= 1) hipLaunchKernelGGL(select_topk_kernel<1>, grid, block, 0, stream, D, K, scores, out);
    else if (slots <= 4) hipLaunchKernelGGL(select_topk_kernel<4>, grid, block, 0, stream, D, K, scores, out);
    else if (slots <= 16) hipLaunchKernelGGL(select_topk_kernel<16>, grid, block, 0, stream, D, K, scores, out);
    else hipLaunchKernelGGL(select_topk_kernel<kSelectMaxSlots>, grid, block, 0, stream, D, K, scores, out);
    return hipGetLastError();
}

}  // namespace dd
