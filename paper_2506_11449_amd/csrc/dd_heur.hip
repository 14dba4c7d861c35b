// Heuristic update of the set of active diagonals (DiagHeur, appendix "Details of the Heuristics-Based
// Method"): the diagonals of lowest magnitude leave, as many inactive candidates enter at random.  The random
// scores are an input, so the result is a pure function of its arguments.
//
// The update is two hard TopK selections (Sec. 3.2, dd_select_block.h) on keys over the D candidates, by one workgroup that
// keeps them in registers:
//   1. key of the magnitude of the active diagonal with offset i (a NaN magnitude counts as -1, below every true
//      magnitude, which is a sum of absolute values), of -inf where no diagonal is active;
//      keep = TopK(K - n_drop)                               the diagonals that stay
//   2. key of +inf for i in keep, of random[i] for i that was not active (finite by contract; NaN counts as -inf), and of
//      NaN -- the lowest rank there is -- for the diagonals that have just left;
//      new = TopK(K)                                         the K - n_drop kept ones and the n_drop grown ones
// Both selections order equal scores by lower index and NaN lowest, and emit ascending indices.
// Bound by latency (one workgroup, two trips to memory, two selections): D = 3072, K = 307 10.5 us in one launch, where five
// launches (table, selection, scores, selection, sources) took 33 us one after the other.  Beyond 16384 candidates the 256
// words that a thread holds do not fit its registers: 135-175 us at 16385 (the five launches 149-173), 218-288 us at 65536
// (571-655), with 10 and 90 % of the candidates active.
#include "dd_common.h"
#include "dd_launch.h"
#include "dd_select_block.h"

#include <float.h>
#include <math.h>

namespace dd {

constexpr int kHeurThreads = 256;

// magnitudes[k] = sum_p |values[k][p]|: one workgroup per diagonal, fixed-order tree reduction
template <typename Tr>
__global__ __launch_bounds__(kHeurThreads) void diag_magnitude_kernel(int L, const typename Tr::storage *__restrict__ values,
                                                                      float *__restrict__ magnitudes)
{
    __shared__ float part[kHeurThreads];
    const typename Tr::storage *row = values + size_t(blockIdx.x) * L;
    float s = 0.f;
    for (int p = threadIdx.x; p < L; p += kHeurThreads) s += fabsf(Tr::load(row + p));
    part[threadIdx.x] = s;
    __syncthreads();
    for (int w = kHeurThreads / 2; w > 0; w >>= 1) {
        if (threadIdx.x < w) part[threadIdx.x] += part[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) magnitudes[blockIdx.x] = part[0];
}

// One workgroup.  slot: table offset -> position in `offsets` (-1: not active), D entries in LDS or, for more candidates
// than fit there, in the caller's scratch.
template <int THREADS, int SLOTS, bool TABLE_IN_LDS>
__global__ __launch_bounds__(THREADS) void heur_update_kernel(int D, int K, int n_keep,
                                                                     const int *__restrict__ offsets,
                                                                     const float *__restrict__ magnitudes,
                                                                     const float *__restrict__ random,
                                                                     int *__restrict__ new_offsets,
                                                                     int *__restrict__ source, int *__restrict__ table)
{
    extern __shared__ int lds_table[];
    __shared__ __attribute__((aligned(16))) SelectScratch<THREADS, SLOTS> scratch;
    int *slot = TABLE_IN_LDS ? lds_table : table;
    const int tid = threadIdx.x;
    float r[SLOTS];  // requested first: needed last
#pragma unroll
    for (int j = 0; j < SLOTS; ++j) r[j] = random[min(j * THREADS + tid, D - 1)];
    for (int i = tid; i < D; i += THREADS) slot[i] = -1;
    __syncthreads();  // one workgroup: its own writes above are ordered before those below
    for (int k = tid; k < K; k += THREADS) slot[canonical_offset(offsets[k], D)] = k;
    __syncthreads();
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

template <int THREADS, int SLOTS, bool TABLE_IN_LDS>
static hipError_t launch_heur(int D, int K, int n_keep, const int *offsets, const float *magnitudes, const float *random,
                              int *new_offsets, int *source, void *ws, hipStream_t stream)
{
    const int lds = TABLE_IN_LDS ? SLOTS * THREADS * int(sizeof(int)) : 0;
    static std::atomic<uint64_t> lds_allowed{0};  // one bit per device
    if (lds)
        if (hipError_t e = allow_dynamic_lds(reinterpret_cast<const void *>(&heur_update_kernel<THREADS, SLOTS, TABLE_IN_LDS>), lds, lds_allowed)) return e;
    hipLaunchKernelGGL((heur_update_kernel<THREADS, SLOTS, TABLE_IN_LDS>), dim3(1), dim3(THREADS), lds, stream, D, K, n_keep, offsets,
                       magnitudes, random, new_offsets, source, static_cast<int *>(ws));
    return hipGetLastError();
}

// Threads as for one score vector (select_threads: what a pass costs grows with the waves that meet at its barrier): 128
// candidates 6.6 us with 1024 threads, 4.6 with 256, 768 7.1 and 6.5, 2048 10 and 9.4.
hipError_t launch_diagheur_update(int D, int K, int n_drop, const int *offsets, const float *magnitudes,
                                  const float *random, int *new_offsets, int *source, void *ws, hipStream_t stream)
{
    const int n_keep = K - n_drop;
    if (select_threads(1, D) == kSelectThreadsFew) {
        constexpr int kFew = kSelectThreadsFew;
        const int slots = (D + kFew - 1) / kFew;
        if (slots <= 1) return launch_heur<kFew, 1, true>(D, K, n_keep, offsets, magnitudes, random, new_offsets, source, ws, stream);
        if (slots <= 4) return launch_heur<kFew, 4, true>(D, K, n_keep, offsets, magnitudes, random, new_offsets, source, ws, stream);
        return launch_heur<kFew, 8, true>(D, K, n_keep, offsets, magnitudes, random, new_offsets, source, ws, stream);
    }
    const int slots = (D + kSelectThreads - 1) / kSelectThreads;
    if (slots <= 4) return launch_heur<kSelectThreads, 4, true>(D, K, n_keep, offsets, magnitudes, random, new_offsets, source, ws, stream);
    if (slots <= 16) return launch_heur<kSelectThreads, 16, true>(D, K, n_keep, offsets, magnitudes, random, new_offsets, source, ws, stream);
    return launch_heur<kSelectThreads, kSelectMaxSlots, false>(D, K, n_keep, offsets, magnitudes, random, new_offsets, source, ws, stream);
}

}  // namespace dd
