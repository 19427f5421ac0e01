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

}  // namespace hbmg
