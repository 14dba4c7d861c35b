// The hard TopK selection (Sec. 3.2, Eq. 4) as a workgroup-level routine, shared by the selection kernel and by
// kernels that select and go on with the result.
//
// Method: scores are mapped to 32-bit keys whose unsigned order is the required total order (NaN lowest, -0 == +0) and
// stay in registers: slot j of thread t is candidate j * THREADS + t.  A four-pass byte-wise radix search finds the K-th
// largest key tau and how many of the keys equal to tau still belong to the selection (the lowest-indexed ones); each
// pass is one LDS histogram behind one barrier, searched by every wave for itself (lane shuffles), so that nothing has to
// be broadcast.  The chosen candidates' places in ascending order come from ballots and a prefix sum over the
// (slot, wave) pairs, which run through the candidates in index order.
//
// What bounds it is latency: one trip to memory for the scores, then a chain of seven barriers; nothing else runs on the
// chip meanwhile.  The first pass, whose byte is the sign and most of the exponent, has few busy counters -- a quarter to half of
// all scores meet at one, 2.6 clk each -- and so counts into four copies by lane (from three candidates per thread on; with two
// and eight copies the shorter vectors are slower).  Measured (graph replay, against one copy and instances for 1, 2, 4, 8, 16
// candidates per thread): one vector of 768 scores 3.9 -> 3.7 us, 3072 5.7 -> 5.0, 4096 6.2 -> 5.5, 8192 12.0 -> 7.3, 16384
// 14.1 -> 11.1; 600 x 768 5.0 -> 4.5, 1000 x 4096 13.6 -> 10.9.
#pragma once
#include "dd_common.h"

namespace dd {

constexpr int kSelectThreads = 1024;   // threads of the kernels that work on score vectors ...
constexpr int kSelectThreadsFew = 256; // ... or these: select_threads
constexpr int kSelectMaxSlots = 64;    // 65536 candidates

// Threads of the workgroup for one score vector, for the selection and for the weights.  Alone on the chip a long vector is done
// sooner by many threads; of many vectors more fit a CU at a time with few, and a short one leaves the other waves waiting at
// barriers.  us with 256 and 1024 threads: selection of 1 x 1024 scores 3.8 and 4.2, 1 x 2048 4.7 and 4.8, 1 x 2304 6.7 and 4.8,
// 600 x 768 4.5 and 7.8, 4000 x 4096 30 and 48; with the weights 1 x 768 4.4 and 5.3, 1 x 2000 6.0 and 6.4, 1 x 3072 9.2 and 6.6,
// 1000 x 4096 18 and 21; weights alone 1 x 64 2.5 and 2.7, 1 x 2000 3.1 and 3.5, 1 x 4096 3.6 and 3.6.
inline bool many_vectors(int batch, int D) { return batch > 256 && D <= 16 * kSelectThreadsFew; }
inline int select_threads(int batch, int D) { return D <= 8 * kSelectThreadsFew || many_vectors(batch, D) ? kSelectThreadsFew : kSelectThreads; }

__device__ __forceinline__ uint32_t score_key(float s)
{
    if (s != s) return 0u;             // NaN: below every number
    uint32_t u = __float_as_uint(s + 0.0f);  // -0 + 0 = +0
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Inclusive prefix sum over the 64 lanes of a wave, without a trip through LDS: four shift-and-add steps inside
// each row of 16 lanes (DPP row_shr, lanes shifted in from outside the row read 0), then the totals of the rows
// before a lane's own row, read from lanes 15, 31 and 47.
__device__ __forceinline__ unsigned wave_inclusive_scan(unsigned v, int lane)
{
#define DD_ROW_SHR(n_) unsigned(__builtin_amdgcn_update_dpp(0, int(v), 0x110 + (n_), 0xf, 0xf, true))
    v += DD_ROW_SHR(1);
    v += DD_ROW_SHR(2);
    v += DD_ROW_SHR(4);
    v += DD_ROW_SHR(8);
#undef DD_ROW_SHR
    const unsigned r0 = unsigned(__builtin_amdgcn_readlane(int(v), 15));
    const unsigned r1 = unsigned(__builtin_amdgcn_readlane(int(v), 31));
    const unsigned r2 = unsigned(__builtin_amdgcn_readlane(int(v), 47));
    const int row = lane >> 4;
    return v + (row >= 1 ? r0 : 0u) + (row >= 2 ? r1 : 0u) + (row >= 3 ? r2 : 0u);
}

template <int THREADS, int SLOTS>
struct SelectScratch {
    static constexpr int kWaves = THREADS / 64, kPairs = SLOTS * kWaves;
    static constexpr int kCopies = SLOTS >= 3 ? 4 : 1, kCopyStride = 264;  // of the first pass's histogram: other banks, rows of 16 bytes
    static constexpr int kCounters = kCopies * kCopyStride + 3 * 256;      // then those of the other passes
    unsigned hist[kCounters];
    unsigned gt[kPairs], eq[kPairs];  // per (slot, wave): how many are larger than tau / equal to it; then those before
};

// Of the D candidates (D <= THREADS * SLOTS) the K with the largest keys, 1 <= K <= D.  place[j]: the position of this
// thread's candidate j * THREADS + threadIdx.x among the chosen ones, ascending by index, or -1.  A workgroup may call it
// again on the same scratch after a barrier.  Groups of THREADS threads of one workgroup may call it side by side, each with keys and
// scratch of its own; tid is then the thread's number within its group.
// MASKED_OUT: many of the candidates may share the lowest keys (-infinity and NaN, what candidates are masked out with); the first
// pass counts these by the wave, where one by one all 64 lanes would wait for the same counter (2765 of 3072: 3 us).
template <int THREADS, int SLOTS, bool MASKED_OUT = false>
__device__ __forceinline__ void select_block(int D, int K, const uint32_t (&key)[SLOTS], SelectScratch<THREADS, SLOTS> &s,
                                             int (&place)[SLOTS], const int tid = int(threadIdx.x))
{
    using Scratch = SelectScratch<THREADS, SLOTS>;
    constexpr int kWaves = Scratch::kWaves, kPairs = Scratch::kPairs;
    const int lane = tid & 63, wave = tid >> 6;
    constexpr int kCopies = Scratch::kCopies, kCopyStride = Scratch::kCopyStride;
    for (int i = tid; i < Scratch::kCounters; i += THREADS) s.hist[i] = 0u;
    __syncthreads();
    unsigned prefix = 0u, mask = 0u, remaining = unsigned(K);
#pragma unroll
    for (int pass = 0; pass < 4; ++pass) {
        const int shift = 24 - 8 * pass;
        unsigned *const hist = s.hist + (pass == 0 ? 0 : kCopies * kCopyStride + (pass - 1) * 256);
        unsigned lowest = 0u;
#pragma unroll
        for (int j = 0; j < SLOTS; ++j) {
            bool counts = j * THREADS + tid < D && (key[j] & mask) == prefix;
            if (MASKED_OUT && pass == 0) {
                const unsigned long long low = __ballot(counts && key[j] >> 24 == 0u);
                lowest += unsigned(__popcll(low));
                counts = counts && key[j] >> 24 != 0u;
            }
            const int copy = pass == 0 ? (lane & (kCopies - 1)) * kCopyStride : 0;
            if (counts) atomicAdd(&hist[copy + ((key[j] >> shift) & 255u)], 1u);
        }
        if (MASKED_OUT && pass == 0 && lane == 0 && lowest) atomicAdd(&hist[0], lowest);
        __syncthreads();
        // lane l owns bins 255 - 4l ... 252 - 4l (descending); the bin where the running count of larger-or-equal keys
        // first reaches `remaining`
        uint4 bins = *reinterpret_cast<const uint4 *>(&hist[252 - 4 * lane]);
        if (pass == 0) {
#pragma unroll
            for (int c = 1; c < kCopies; ++c) {
                const uint4 more = *reinterpret_cast<const uint4 *>(&hist[c * kCopyStride + 252 - 4 * lane]);
                bins.x += more.x, bins.y += more.y, bins.z += more.z, bins.w += more.w;
            }
        }
        const unsigned h[4] = {bins.w, bins.z, bins.y, bins.x};
        const unsigned mine = h[0] + h[1] + h[2] + h[3];
        const unsigned incl = wave_inclusive_scan(mine, lane);
        unsigned above = incl - mine;  // keys in bins larger than this lane's
        unsigned bin = unsigned(255 - 4 * lane);
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const bool next = above + h[i] < remaining && bin + unsigned(i) == unsigned(255 - 4 * lane);
            above += next ? h[i] : 0u;
            bin -= next ? 1u : 0u;
        }
        const int owner = __ffsll(__ballot(incl >= remaining)) - 1;  // the first lane that reaches it
        remaining -= unsigned(__builtin_amdgcn_readlane(int(above), owner));  // still to take inside the chosen bin
        prefix |= unsigned(__builtin_amdgcn_readlane(int(bin), owner)) << shift;
        mask |= 255u << shift;
    }
    const uint32_t tau = prefix;         // the K-th largest key
    const unsigned take_eq = remaining;  // how many keys equal to tau are selected (>= 1)
#pragma unroll
    for (int j = 0; j < SLOTS; ++j) {
        const bool in = j * THREADS + tid < D;
        const unsigned long long gt = __ballot(in && key[j] > tau), eq = __ballot(in && key[j] == tau);
        if (lane == 0) {
            s.gt[j * kWaves + wave] = unsigned(__popcll(gt));
            s.eq[j * kWaves + wave] = unsigned(__popcll(eq));
        }
    }
    __syncthreads();
    if (wave == 0) {  // pairs before each pair, in index order
        constexpr int kOwn = (kPairs + 63) / 64;
        unsigned sum_gt = 0u, sum_eq = 0u;
#pragma unroll
        for (int i = 0; i < kOwn; ++i) {
            const int e = lane * kOwn + i;
            sum_gt += e < kPairs ? s.gt[e] : 0u;
            sum_eq += e < kPairs ? s.eq[e] : 0u;
        }
        unsigned before_gt = wave_inclusive_scan(sum_gt, lane) - sum_gt, before_eq = wave_inclusive_scan(sum_eq, lane) - sum_eq;
#pragma unroll
        for (int i = 0; i < kOwn; ++i) {
            const int e = lane * kOwn + i;
            if (e < kPairs) {
                const unsigned g = s.gt[e], q = s.eq[e];
                s.gt[e] = before_gt;
                s.eq[e] = before_eq;
                before_gt += g;
                before_eq += q;
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < SLOTS; ++j) {
        const bool in = j * THREADS + tid < D;
        const bool is_gt = in && key[j] > tau, is_eq = in && key[j] == tau;
        const unsigned long long gt = __ballot(is_gt), eq = __ballot(is_eq);
        const unsigned before_gt = s.gt[j * kWaves + wave] + __builtin_amdgcn_mbcnt_hi(unsigned(gt >> 32), __builtin_amdgcn_mbcnt_lo(unsigned(gt), 0u));
        const unsigned before_eq = s.eq[j * kWaves + wave] + __builtin_amdgcn_mbcnt_hi(unsigned(eq >> 32), __builtin_amdgcn_mbcnt_lo(unsigned(eq), 0u));
        place[j] = is_gt || (is_eq && before_eq < take_eq) ? int(before_gt + min(before_eq, take_eq)) : -1;
    }
}

// The same for scores that the threads hold (slot j of thread t: candidate j * THREADS + t, anything past the end); the chosen
// indices go to `dst` (global or LDS), ascending.  Ends without a barrier.
template <int THREADS, int SLOTS>
__device__ __forceinline__ void select_held_block(int D, int K, const float (&a)[SLOTS], SelectScratch<THREADS, SLOTS> &s, int *dst)
{
    uint32_t key[SLOTS];
    int place[SLOTS];
#pragma unroll
    for (int j = 0; j < SLOTS; ++j) key[j] = score_key(a[j]);
    select_block<THREADS, SLOTS>(D, K, key, s, place);
#pragma unroll
    for (int j = 0; j < SLOTS; ++j)
        if (place[j] >= 0) dst[place[j]] = j * THREADS + int(threadIdx.x);
}
// The same from a vector of scores in memory.
template <int THREADS, int SLOTS>
__device__ __forceinline__ void select_topk_block(int D, int K, const float *__restrict__ row,
                                                  SelectScratch<THREADS, SLOTS> &s, int *dst)
{
    float a[SLOTS];
#pragma unroll
    for (int j = 0; j < SLOTS; ++j) a[j] = row[min(j * THREADS + int(threadIdx.x), D - 1)];
    select_held_block<THREADS, SLOTS>(D, K, a, s, dst);
}

}  // namespace dd
