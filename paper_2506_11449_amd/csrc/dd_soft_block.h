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
template <bool MAX, int THREADS>
__device__ __forceinline__ float block_reduce(float v, float *scratch /* [THREADS / 64] */)
{
    constexpr int kWaves = THREADS / 64;
    v = MAX ? wave_max(v) : wave_sum(v);
    __syncthreads();  // scratch may still be read from a previous reduction
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

// v[j] += value(i) (or the larger) over a thread's candidates of part j, the first P of its N parts side by side: past the end
// the last candidate once more, and dropped
template <bool MAX, int THREADS, int P, int N, class Value>
__device__ __forceinline__ void add_parts(int D, float (&v)[N], Value value)
{
    for (int first = threadIdx.x; first < D; first += kSoftLanes * kSoftParts)
#pragma unroll
        for (int j = 0; j < P; ++j) {
            const int i = first + j * THREADS;
            const float x = value(min(i, D - 1));
            v[j] = i < D ? (MAX ? fmaxf(v[j], x) : v[j] + x) : v[j];
        }
}

// value(i) of the D candidates, summed (or the largest) over the workgroup
template <bool MAX, int THREADS, class Value>
__device__ __forceinline__ float reduce_scores(int D, SoftScratch &s, Value value)
{
    static_assert(THREADS == kSoftLanes || THREADS == kSoftLanes * kSoftParts, "a thread holds a lane or one part of it");
    constexpr int N = kSoftLanes * kSoftParts / THREADS;
    float v[N];
#pragma unroll
    for (int j = 0; j < N; ++j) v[j] = MAX ? -INFINITY : 0.f;
    if (N > 1 && D <= 3 * THREADS) {  // one round of fewer parts
        if (D <= THREADS) add_parts<MAX, THREADS, 1>(D, v, value);
        else if (D <= 2 * THREADS) add_parts<MAX, THREADS, N < 2 ? N : 2>(D, v, value);
        else add_parts<MAX, THREADS, N < 3 ? N : 3>(D, v, value);
    } else {
        add_parts<MAX, THREADS, N>(D, v, value);
    }
    if constexpr (MAX) {
#pragma unroll
        for (int j = 1; j < N; ++j) v[0] = fmaxf(v[0], v[j]);
        return block_reduce<true, THREADS>(v[0], s.waves);
    } else if constexpr (N == kSoftParts) {
        return block_reduce<false, THREADS>((v[0] + v[1]) + (v[2] + v[3]), s.waves);
    } else {
        s.parts[threadIdx.x / kSoftLanes][threadIdx.x % kSoftLanes] = v[0];  // last read two barriers ago
        __syncthreads();
        const int lane = threadIdx.x % kSoftLanes;
        return block_reduce<false, kSoftLanes>((s.parts[0][lane] + s.parts[1][lane]) + (s.parts[2][lane] + s.parts[3][lane]), s.waves);
    }
}

// alpha_tilde_i = min(K * exp((a_i - max) / temp) / sum_j exp((a_j - max) / temp), 1)
template <int THREADS>
__device__ __forceinline__ void soft_topk_block(int D, float k_over_1, float inv_temp, const float *__restrict__ a,
                                                float *__restrict__ out)
{
    __shared__ SoftScratch scratch;
    const float m = reduce_scores<true, THREADS>(D, scratch, [&](int i) { return a[i]; });
    const float s = reduce_scores<false, THREADS>(D, scratch, [&](int i) { return expf((a[i] - m) * inv_temp); });
    const float scale = k_over_1 / s;
    for (int i = threadIdx.x; i < D; i += THREADS) out[i] = fminf(scale * expf((a[i] - m) * inv_temp), 1.f);
}

}  // namespace dd
