// Arithmetic on the row boundaries of a schedule, for the planning kernels and for host code that checks it.  Offsets come from the
// caller's device memory and cannot be checked before a launch, so whatever they hold, a group lies in [0, M] and a sum of
// groups never passes M (nor wraps: 65 536 groups that each claim all of M rows are far more than 2^31).
#pragma once
#include <stdint.h>

#ifdef __HIPCC__
#define MOE_ROWS_FN __host__ __device__ __forceinline__
#else
#define MOE_ROWS_FN inline
#endif

// rows of group g and its first row: [offsets[g], offsets[g + 1]) clamped to [0, M] and to non-decreasing order
MOE_ROWS_FN int group_rows(const int32_t* offsets, int g, int M, int& lo) {
    int a = offsets[g], b = offsets[g + 1];
    a = a < 0 ? 0 : (a > M ? M : a);
    b = b < a ? a : (b > M ? M : b);
    lo = a;
    return b - a;
}

// first row of the first group
MOE_ROWS_FN int first_row(const int32_t* offsets, int M) { const int a = offsets[0]; return a < 0 ? 0 : (a > M ? M : a); }

// a + b, at most M (0 <= a, b <= M < 2^31)
MOE_ROWS_FN int add_rows(int a, int b, int M) {
    const unsigned int sum = (unsigned int)a + (unsigned int)b;
    return (int)(sum < (unsigned int)M ? sum : (unsigned int)M);
}
