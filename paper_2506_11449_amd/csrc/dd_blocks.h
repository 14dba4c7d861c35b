// Which 32 x 16 blocks of the dense operand a diagonal crosses, from a bitmap of the active offsets in LDS.
#pragma once
#include "dd_common.h"

namespace dd {

constexpr int kBlkMaxD = 8192;

// Bit i of the result: is offset lo + i (mod D) active?  bits: one bit per candidate, D a multiple of 128; -2 D <= lo < D.
__device__ __forceinline__ unsigned long long blk_window(const unsigned *bits, int D, int lo)
{
    lo += lo < 0 ? D : 0;
    lo += lo < 0 ? D : 0;
    const int words = D >> 5;
    int w = lo >> 5;
    const int s = lo & 31;
    const unsigned w0 = bits[w];
    w = w + 1 == words ? 0 : w + 1;
    const unsigned w1 = bits[w];
    w = w + 1 == words ? 0 : w + 1;
    const unsigned w2 = bits[w];
    const unsigned long long window = (((unsigned long long)w1 << 32) | w0) >> s;  // 64 - s >= 33 bits
    return s ? window | (unsigned long long)w2 << (64 - s) : window;
}

// Is any of the 47 offsets lo, lo+1, ..., lo+46 (mod D) active?
__device__ __forceinline__ bool blk_crossed(const unsigned *bits, int D, int lo) { return (blk_window(bits, D, lo) & ((1ull << 47) - 1)) != 0; }

// The first of the 47 offsets (long - short index) that run through the block of output columns j0 ... j0 + 31 and
// contraction indices i0 ... i0 + 15; long_cols: the columns are the long side.
__device__ __forceinline__ int blk_first_offset(int j0, int i0, bool long_cols) { return long_cols ? j0 - i0 - 15 : i0 - j0 - 31; }

}  // namespace dd
