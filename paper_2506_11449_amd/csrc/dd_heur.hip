// Heuristic update of the set of active diagonals (DiagHeur, appendix "Details of the Heuristics-Based
// Method"): the diagonals of lowest magnitude leave, as many inactive candidates enter at random.  The random
// scores are an input, so the result is a pure function of its arguments.
//
// The update is two hard TopK selections (Sec. 3.2, dd_select_block.h) on keys over the D candidates, by one workgroup that
// keeps them in registers (up to 4096 candidates side by side: heur_update_pair_kernel):
//   1. key of the magnitude of the active diagonal with offset i (a NaN magnitude counts as -1, below every true
//      magnitude, which is a sum of absolute values), of -inf where no diagonal is active;
//      keep = TopK(K - n_drop)                               the diagonals that stay
//   2. key of +inf for i in keep, of random[i] for i that was not active (finite by contract; NaN counts as -inf), and of
//      NaN -- the lowest rank there is -- for the diagonals that have just left;
//      new = TopK(K)                                         the K - n_drop kept ones and the n_drop grown ones
// Both selections order equal scores by lower index and NaN lowest, and emit ascending indices.
// Bound by latency (one workgroup, two trips to memory, the barriers of the selections and the LDS atomics of their first passes).
// Beyond 16384 candidates the 256 words that a thread holds do not fit its registers: 135-175 us at 16385 (five launches -- table,
// selection, scores, selection, sources -- 149-173), 218-288 us at 65536 (571-655), with 10 and 90 % of the candidates active.
#include "dd_common.h"
#include "dd_launch.h"
#include "dd_select_block.h"

#include <float.h>
#include <math.h>

namespace dd {

constexpr int kHeurThreads = 256;

// magnitudes[k] = sum_p |values[k][p]|: one workgroup per diagonal, fixed-order tree reduction (thread t's sum over p = t, t + 256, ...;
// then t with t + 128, t + 64, ... t + 1).  Bound by latency: eight values are requested
// at a time, and after one barrier a wave adds by lane shuffles (307 diagonals of 768 bf16 values 3.05 -> 2.94 us, 1638 of 4096 4.63 -> 4.54).
template <typename Tr>
__global__ __launch_bounds__(kHeurThreads) void diag_magnitude_kernel(int L, const typename Tr::storage *__restrict__ values,
                                                                      float *__restrict__ magnitudes)
{
    __shared__ float part[kHeurThreads];
    const typename Tr::storage *row = values + size_t(blockIdx.x) * L;
    float s = 0.f;
    for (int first = threadIdx.x; first < L; first += 8 * kHeurThreads) {
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u)
            v[u] = first + u * kHeurThreads < L ? fabsf(Tr::load(row + first + u * kHeurThreads)) : 0.f;
#pragma unroll
        for (int u = 0; u < 8; ++u) s += v[u];
    }
    part[threadIdx.x] = s;
    __syncthreads();
    if (threadIdx.x >= 64) return;
    s = (s + part[threadIdx.x + 128]) + (part[threadIdx.x + 64] + part[threadIdx.x + 192]);
#pragma unroll
    for (int w = 32; w > 0; w >>= 1) s += __shfl_down(s, w, 64);
    if (threadIdx.x == 0) magnitudes[blockIdx.x] = s;
}

// The two selections one after the other, as above.  slot: table offset -> position in `offsets` (-1: not active), complete.
template <int THREADS, int SLOTS>
__device__ __forceinline__ void heur_in_turn(int D, int K, int n_keep, const int *slot, const float *__restrict__ magnitudes,
                                             const float *__restrict__ random, int *__restrict__ new_offsets, int *__restrict__ source,
                                             SelectScratch<THREADS, SLOTS> &scratch)
{
    const int tid = threadIdx.x;
    float r[SLOTS];  // requested first: needed last
#pragma unroll
    for (int j = 0; j < SLOTS; ++j) r[j] = random[min(j * THREADS + tid, D - 1)];
    int mine[SLOTS], place[SLOTS];
    uint32_t key[SLOTS];
#pragma unroll
    for (int j = 0; j < SLOTS; ++j) {
        mine[j] = slot[min(j * THREADS + tid, D - 1)];
        const float m = mine[j] >= 0 ? magnitudes[mine[j]] : -INFINITY;
        key[j] = score_key(m != m ? -1.f : m);
        place[j] = -1;
    }
    if (n_keep > 0) {
        select_block<THREADS, SLOTS, true>(D, n_keep, key, scratch, place);
        __syncthreads();
    }
#pragma unroll
    for (int j = 0; j < SLOTS; ++j) {
        const float grow = r[j] != r[j] ? -INFINITY : r[j];
        key[j] = score_key(place[j] >= 0 ? INFINITY : (mine[j] >= 0 ? NAN : grow));
    }
    select_block<THREADS, SLOTS>(D, K, key, scratch, place);
#pragma unroll
    for (int j = 0; j < SLOTS; ++j)
        if (place[j] >= 0) {
            new_offsets[place[j]] = j * THREADS + tid;
            source[place[j]] = mine[j];
        }
}

// One workgroup for more candidates than two groups of threads hold.  table: D entries of the caller's scratch, or null (in LDS).
template <int SLOTS>
__global__ __launch_bounds__(kSelectThreads) void heur_update_kernel(int D, int K, int n_keep, const int *__restrict__ offsets,
                                                                     const float *__restrict__ magnitudes,
                                                                     const float *__restrict__ random,
                                                                     int *__restrict__ new_offsets,
                                                                     int *__restrict__ source, int *__restrict__ table)
{
    extern __shared__ int lds_table[];
    __shared__ __attribute__((aligned(16))) SelectScratch<kSelectThreads, SLOTS> scratch;
    int *slot = SLOTS < kSelectMaxSlots ? lds_table : table;
    for (int i = threadIdx.x; i < D; i += kSelectThreads) slot[i] = -1;
    __syncthreads();  // one workgroup: its own writes above are ordered before those below
    for (int k = threadIdx.x; k < K; k += kSelectThreads) slot[canonical_offset(offsets[k], D)] = k;
    __syncthreads();
    heur_in_turn<kSelectThreads, SLOTS>(D, K, n_keep, slot, magnitudes, random, new_offsets, source, scratch);
}

// Both selections side by side.  The second one chooses n_drop of the candidates that were not active, whichever diagonals stay:
// its +inf are the first one's result, and its NaN never chosen (n_drop <= D - K).  So a group of threads selects the diagonals that stay
// while another selects those that enter, through the same seven barriers; the places in the union come from the words of chosen
// candidates.  Arguments outside the contract that this would answer otherwise -- a random score of +inf, offsets given twice or
// magnitudes of -inf that let an inactive candidate stay -- are noticed, and done in turn.
// A group has 256 threads up to 1024 candidates, then 512, and no more slots than it needs (a slot costs 0.7 us).  Against one selection
// after the other by 256 threads (from 2049 candidates on 1024), graph replay, us: 256 candidates 4.8 -> 4.4, 768 6.7 -> 5.5, 2048 9.7 -> 7.5, 3072
// (307 active) 11.3 -> 9.0, 4096 (205) 11.9 -> 10.4.
template <int THREADS, int SLOTS>  // of a group
__global__ __launch_bounds__(2 * THREADS) void heur_update_pair_kernel(int D, int K, int n_keep, const int *__restrict__ offsets,
                                                                       const float *__restrict__ magnitudes,
                                                                       const float *__restrict__ random, int *__restrict__ new_offsets,
                                                                       int *__restrict__ source)
{
    constexpr int kWaves = THREADS / 64, kWords = SLOTS * kWaves, kTurnSlots = (SLOTS + 1) / 2;
    static_assert(kWords <= 64, "a word for each lane");
    extern __shared__ int slot[];  // offset -> position in `offsets`, -1: not active
    union Scratch {
        SelectScratch<THREADS, SLOTS> pair[2];
        SelectScratch<2 * THREADS, kTurnSlots> turn;
    };
    __shared__ __attribute__((aligned(16))) Scratch scratch;
    __shared__ unsigned long long chosen[2][kWords];
    __shared__ int in_turn;
    const int group = __builtin_amdgcn_readfirstlane(int(threadIdx.x) / THREADS), tid = int(threadIdx.x) - group * THREADS;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool stays = group == 0;
    float score[SLOTS];
    if (!stays) {  // requested first
#pragma unroll
        for (int j = 0; j < SLOTS; ++j) score[j] = random[min(j * THREADS + tid, D - 1)];
    }
    for (int i = threadIdx.x; i < D; i += 2 * THREADS) slot[i] = -1;
    if (threadIdx.x == 0) in_turn = 0;
    __syncthreads();
    for (int k = threadIdx.x; k < K; k += 2 * THREADS) slot[canonical_offset(offsets[k], D)] = k;
    __syncthreads();
    int mine[SLOTS], place[SLOTS];
    uint32_t key[SLOTS];
#pragma unroll
    for (int j = 0; j < SLOTS; ++j) {
        mine[j] = slot[min(j * THREADS + tid, D - 1)];
        if (stays) {
            const float m = mine[j] >= 0 ? magnitudes[mine[j]] : -INFINITY;
            key[j] = score_key(m != m ? -1.f : m);
        } else {
            if (mine[j] < 0 && score[j] == INFINITY) in_turn = 1;
            key[j] = score_key(mine[j] >= 0 ? NAN : (score[j] != score[j] ? -INFINITY : score[j]));
        }
    }
    const int count = stays ? n_keep : K - n_keep;
    select_block<THREADS, SLOTS, true>(D, max(count, 1), key, scratch.pair[group], place, tid);
#pragma unroll
    for (int j = 0; j < SLOTS; ++j) {
        const unsigned long long word = __ballot(place[j] >= 0 && count > 0);
        if (lane == 0) chosen[group][j * kWaves + wave] = word;
        if (place[j] >= 0 && count > 0 && stays == (mine[j] < 0)) in_turn = 1;
    }
    __syncthreads();
    if (in_turn) {
        heur_in_turn<2 * THREADS, kTurnSlots>(D, K, n_keep, slot, magnitudes, random, new_offsets, source, scratch.turn);
        return;
    }
    const unsigned long long own = lane < kWords ? chosen[0][lane] | chosen[1][lane] : 0ull;
    const unsigned in_word = unsigned(__popcll(own)), before = wave_inclusive_scan(in_word, lane) - in_word;
#pragma unroll
    for (int j = 0; j < SLOTS; ++j) {
        const int w = j * kWaves + wave;
        const unsigned lo = unsigned(__builtin_amdgcn_readlane(int(unsigned(own)), w)), hi = unsigned(__builtin_amdgcn_readlane(int(own >> 32), w));
        const unsigned at = unsigned(__builtin_amdgcn_readlane(int(before), w)) + __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0u));
        if (place[j] >= 0 && count > 0) {
            new_offsets[at] = j * THREADS + tid;
            source[at] = mine[j];
        }
    }
}

hipError_t launch_diag_magnitude(int K, int L, bool bf16, const void *values, float *magnitudes, hipStream_t stream)
{
    if (bf16)
        hipLaunchKernelGGL(diag_magnitude_kernel<BF16>, dim3(K), dim3(kHeurThreads), 0, stream, L,
                           static_cast<const uint16_t *>(values), magnitudes);
    else
        hipLaunchKernelGGL(diag_magnitude_kernel<F32>, dim3(K), dim3(kHeurThreads), 0, stream, L,
                           static_cast<const float *>(values), magnitudes);
    return hipGetLastError();
}

size_t diagheur_ws_bytes(int D, int K)
{
    // two tables of D entries and one of K, each a multiple of 256 bytes (of which the kernel for layers too wide for LDS
    // uses one table)
    auto up = [](size_t b) { return (b + 255) / 256 * 256; };
    return 2 * up(size_t(D) * 4) + up(size_t(K) * 4);
}

template <int SLOTS>
static hipError_t launch_heur(int D, int K, int n_keep, const int *offsets, const float *magnitudes, const float *random,
                              int *new_offsets, int *source, void *ws, hipStream_t stream)
{
    const int lds = SLOTS < kSelectMaxSlots ? SLOTS * kSelectThreads * int(sizeof(int)) : 0;
    static std::atomic<uint64_t> lds_allowed{0};  // one bit per device
    if (lds)
        if (hipError_t e = allow_dynamic_lds(reinterpret_cast<const void *>(&heur_update_kernel<SLOTS>), lds, lds_allowed)) return e;
    hipLaunchKernelGGL(heur_update_kernel<SLOTS>, dim3(1), dim3(kSelectThreads), lds, stream, D, K, n_keep, offsets, magnitudes, random,
                       new_offsets, source, static_cast<int *>(ws));
    return hipGetLastError();
}

template <int THREADS, int SLOTS>
static hipError_t launch_heur_pair(int D, int K, int n_keep, const int *offsets, const float *magnitudes, const float *random,
                                   int *new_offsets, int *source, hipStream_t stream)
{
    hipLaunchKernelGGL((heur_update_pair_kernel<THREADS, SLOTS>), dim3(1), dim3(2 * THREADS), size_t(D) * sizeof(int), stream, D, K, n_keep, offsets,
                       magnitudes, random, new_offsets, source);
    return hipGetLastError();
}

hipError_t launch_diagheur_update(int D, int K, int n_drop, const int *offsets, const float *magnitudes,
                                  const float *random, int *new_offsets, int *source, void *ws, hipStream_t stream)
{
    const int n_keep = K - n_drop;
#define DD_PAIR(threads_, slots_) launch_heur_pair<threads_, slots_>(D, K, n_keep, offsets, magnitudes, random, new_offsets, source, stream)
    if (D <= 256) return DD_PAIR(256, 1);
    if (D <= 512) return DD_PAIR(256, 2);
    if (D <= 768) return DD_PAIR(256, 3);
    if (D <= 1024) return DD_PAIR(256, 4);
    if (D <= 1536) return DD_PAIR(512, 3);
    if (D <= 2048) return DD_PAIR(512, 4);
    if (D <= 3072) return DD_PAIR(512, 6);
    if (D <= 4096) return DD_PAIR(512, 8);
#undef DD_PAIR
    if (D <= 8 * kSelectThreads) return launch_heur<8>(D, K, n_keep, offsets, magnitudes, random, new_offsets, source, ws, stream);
    if (D <= 16 * kSelectThreads) return launch_heur<16>(D, K, n_keep, offsets, magnitudes, random, new_offsets, source, ws, stream);
    return launch_heur<kSelectMaxSlots>(D, K, n_keep, offsets, magnitudes, random, new_offsets, source, ws, stream);
}

}  // namespace dd
