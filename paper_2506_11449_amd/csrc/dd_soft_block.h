// Soft TopK weights of one score vector by one workgroup (Sec. 3.2, Eq. 5), shared by the kernel
// that computes only them and by the selection kernel that also emits them.
#pragma once
#include "dd_common.h"

namespace dd {

// Sums over a score vector have one order whatever the threads of the workgroup: candidate i belongs to part (i / 256) % 4
// of lane i % 256; a lane's four parts are added first, then the lanes.  With 256 threads a thread keeps the parts of a
// lane, with 1024 one of them each.
constexpr int kSoftLanes = 256, kSoftParts = 4;

__device__ __forceinline__ float wave_sum(float v)
{
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
    return v;
}
__device__ __forceinline__ float wave_max(float v)
{
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) v = fmaxf(v, __shfl_xor(v, d, 64));
    return v;
}
// all-reduce over the first THREADS threads of a workgroup; every thread of the workgroup gets the result
template <bool MAX, int THREADS, bool FRESH = false>  // FRESH: no reduction before reads this scratch
__device__ __forceinline__ float block_reduce(float v, float *scratch /* [THREADS / 64] */)
{
    constexpr int kWaves = THREADS / 64;
    v = MAX ? wave_max(v) : wave_sum(v);
    if (!FRESH) __syncthreads();  // scratch may still be read from a previous reduction
    if ((threadIdx.x & 63) == 0 && threadIdx.x < THREADS) scratch[threadIdx.x >> 6] = v;
    __syncthreads();
    float r[kWaves];
#pragma unroll
    for (int w = 0; w < kWaves; ++w) r[w] = scratch[w];
#pragma unroll
    for (int d = kWaves / 2; d >= 1; d /= 2)
#pragma unroll
        for (int w = 0; w < d; ++w) r[w] = MAX ? fmaxf(r[w], r[w + d]) : r[w] + r[w + d];
    return r[0];
}

struct SoftScratch {
    float parts[kSoftParts][kSoftLanes], waves[kSoftLanes * kSoftParts / 64];
};

// value(i) of the D candidates, summed (or the largest) over a workgroup of 1024 threads
template <bool MAX, class Value>
__device__ __forceinline__ float reduce_scores(int D, SoftScratch &s, Value value)
{
    constexpr int THREADS = kSoftLanes * kSoftParts;
    float v = MAX ? -INFINITY : 0.f;
    for (int i = threadIdx.x; i < D; i += THREADS) v = MAX ? fmaxf(v, value(i)) : v + value(i);
    if constexpr (MAX) {
        return block_reduce<true, THREADS>(v, s.waves);
    } else {
        s.parts[threadIdx.x / kSoftLanes][threadIdx.x % kSoftLanes] = v;  // last read two barriers ago
        __syncthreads();
        const int lane = threadIdx.x % kSoftLanes;
        return block_reduce<false, kSoftLanes>((s.parts[0][lane] + s.parts[1][lane]) + (s.parts[2][lane] + s.parts[3][lane]), s.waves);
    }
}

// The same from registers: slot j of thread t holds candidate j * THREADS + t (0 past the end, or -infinity for the largest), which is
// part j % 4 of lane t with 256 threads and part t / 256 of lane t % 256 with 1024.  waves, parts: not used by a reduction before.
template <int THREADS, int SLOTS>
__device__ __forceinline__ float largest_held(const float (&x)[SLOTS], float *waves)
{
    float v = -INFINITY;
#pragma unroll
    for (int j = 0; j < SLOTS; ++j) v = fmaxf(v, x[j]);
    return block_reduce<true, THREADS, true>(v, waves);
}
template <int THREADS, int SLOTS>
__device__ __forceinline__ float sum_held(const float (&x)[SLOTS], float *waves, float (&parts)[kSoftParts][kSoftLanes])
{
    constexpr int N = kSoftLanes * kSoftParts / THREADS;
    float v[N];
#pragma unroll
    for (int j = 0; j < N; ++j) v[j] = 0.f;
#pragma unroll
    for (int j = 0; j < SLOTS; ++j) v[j % N] += x[j];
    if constexpr (N == kSoftParts) {
        return block_reduce<false, THREADS, true>((v[0] + v[1]) + (v[2] + v[3]), waves);
    } else {
        parts[threadIdx.x / kSoftLanes][threadIdx.x % kSoftLanes] = v[0];
        __syncthreads();
        const int lane = threadIdx.x % kSoftLanes;
        return block_reduce<false, kSoftLanes, true>((parts[0][lane] + parts[1][lane]) + (parts[2][lane] + parts[3][lane]), waves);
    }
}
struct HeldScratch {
    float parts[2][kSoftParts][kSoftLanes], waves[3][kSoftLanes * kSoftParts / 64];
};

// e[j] = exp((a_j - max) / temp), 0 past the end; returns their sum
template <int THREADS, int SLOTS>
__device__ __forceinline__ float exponentials_held(int D, float inv_temp, const float (&a)[SLOTS], HeldScratch &s, float (&e)[SLOTS])
{
    float x[SLOTS];
#pragma unroll
    for (int j = 0; j < SLOTS; ++j) x[j] = j * THREADS + int(threadIdx.x) < D ? a[j] : -INFINITY;
    const float m = largest_held<THREADS, SLOTS>(x, s.waves[0]);
#pragma unroll
    for (int j = 0; j < SLOTS; ++j) e[j] = j * THREADS + int(threadIdx.x) < D ? expf((a[j] - m) * inv_temp) : 0.f;
    return sum_held<THREADS, SLOTS>(e, s.waves[1], s.parts[0]);
}

// Candidates that a thread holds at most; longer vectors (from 16385 candidates on) are read again by each pass.  Held, the scores are
// read and their exponentials taken once, us before and now: selection and weights of 1 x 768 5.7 -> 4.4 (with 256 threads, which had been
// behind 1024 while each pass read memory), 1 x 4096 9.1 -> 7.1, 1000 x 4096 24.8 -> 17.9; weights of 1 x 768 3.2 -> 2.7, their derivative 4.0 ->
// 3.0, of 1000 x 4096 29 -> 9.7.  No more are held than a thread has, in steps of a third or so: with room for 16384, 300 x 4467 took 8.7 and
// 13.3 us, behind the 7.3 and 10.4 of passes over memory; 5.9 and 7.1 with room for 6144.
constexpr int kSoftHeldSlots = 16;
// scores of a thread's candidates, the last one once more past the end
template <int THREADS, int SLOTS>
__device__ __forceinline__ void hold(int D, const float *__restrict__ row, float (&a)[SLOTS])
{
#pragma unroll
    for (int j = 0; j < SLOTS; ++j) a[j] = row[min(j * THREADS + int(threadIdx.x), D - 1)];
}

// alpha_tilde_i = min(K * exp((a_i - max) / temp) / sum_j exp((a_j - max) / temp), 1)
template <int THREADS, int SLOTS>
__device__ __forceinline__ void soft_topk_held(int D, float k_over_1, float inv_temp, const float (&a)[SLOTS], float *__restrict__ out)
{
    __shared__ HeldScratch scratch;
    float e[SLOTS];
    const float scale = k_over_1 / exponentials_held<THREADS, SLOTS>(D, inv_temp, a, scratch, e);
#pragma unroll
    for (int j = 0; j < SLOTS; ++j)
        if (j * THREADS + int(threadIdx.x) < D) out[j * THREADS + threadIdx.x] = fminf(scale * e[j], 1.f);
}
// the same with the scores read from memory each time
__device__ __forceinline__ void soft_topk_block(int D, float k_over_1, float inv_temp, const float *__restrict__ a,
                                                float *__restrict__ out)
{
    __shared__ SoftScratch scratch;
    const float m = reduce_scores<true>(D, scratch, [&](int i) { return a[i]; });
    const float s = reduce_scores<false>(D, scratch, [&](int i) { return expf((a[i] - m) * inv_temp); });
    const float scale = k_over_1 / s;
    for (int i = threadIdx.x; i < D; i += kSoftLanes * kSoftParts) out[i] = fminf(scale * expf((a[i] - m) * inv_temp), 1.f);
}

}  // namespace dd
