// What the kernels that keep an input patch in LDS share: the patch height of a
// tile, and divisions by launch constants.
#pragma once
#include "dsq_kernels.h"

#if defined(__HIPCC__)
// x / d for x >= 0 and d >= 1 by multiplication: with m = min(floor(2^32 / d), 2^32 - 1)
// (dsq_division_constant, on the host) the high word of x * m is the quotient or one
// less, so one correction suffices.  Wave-uniform operands stay on the scalar unit.
__device__ __forceinline__ int dsq_idiv(int x, int d, uint32_t m, int &rem)
{
    int q = (int)__umulhi((uint32_t)x, m);
    int r = x - q * d;
    if (r >= d) { ++q; r -= d; }
    rem = r;
    return q;
}
#endif

inline uint32_t dsq_division_constant(int d)
{
    const unsigned long long m = (1ull << 32) / (unsigned long long)d;
    return m > 0xFFFFFFFFull ? 0xFFFFFFFFu : (uint32_t)m;
}

// Patch rows of the worst tile of BP consecutive pixels (a power of two) of a strip of
// TW columns; see conv_patch.hip.
int dsq_patch_rows(const DsqConvArgs &a, int BP, int TW, int row_tiles);
