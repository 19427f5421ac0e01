// bmg_quot.h -- quotients by a diagonal whose reciprocal is at hand.
#pragma once

namespace hbmg {

// r / d with y = 1 / d (rounded to nearest): the product r y and one
// correction by its remainder (Markstein).  With y, r / d and r in the normal
// range the result is the rounded quotient, as the division's (no difference
// in 4e8 random pairs per type); a non-finite r gives NaN.  The three
// dependent operations take the place of a division's eleven, and the
// reciprocal, which depends on no iterate, is off the chain of updates.
template <typename T>
__device__ __forceinline__ T div_by(T r, T d, T y)
{
    const T q = r * y;
    const T e = __builtin_elementwise_fma(-d, q, r);
    return __builtin_elementwise_fma(e, y, q);
}

// Reciprocals of diagonals d, and the entries of a coarse inverse, which grow to
// about 1e4 / d, are finite from here up.  Where a finest diagonal is smaller the
// setup stores the operator times TINY_SCALE, and solves take b times the same:
// a power of two, so the iterates are those of the operator itself.  A smaller
// one serves FP32 copies with diagonals below the normal range of a float.
constexpr double TINY_SCALE = 0x1p80, TINY_SCALE32 = 0x1p64;
__host__ __device__ inline bool tiny_diag(double d) { return d != 0.0 && __builtin_fabs(d) < 0x1p-1000; }

}  // namespace hbmg
