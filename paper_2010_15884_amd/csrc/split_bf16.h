// Numbers of fp32 as exact sums of three bf16 numbers, for the matrix cores (gfx950): v = v1 + v2 + v3, each the rest
// rounded to nearest (8 + 8 + 8 bits: nothing of the 24 is lost).  Six of the nine products of two such numbers are taken --
// x1f1, x1f2, x2f1, x2f2, x1f3, x3f1 -- and accumulated in fp32; the three dropped ones are below 2^-25 of the term and
// of either sign.  bf16 has the exponent range of fp32, so nothing is scaled.  What the split cannot carry has to be looked for in
// every input: infinities, NaN (the zeros of a Toeplitz form would spread them to outputs whose window does not hold
// them), magnitudes from 2^80 on and non-zero ones below split_tiny_limit().
#pragma once

#include <hip/hip_runtime.h>

namespace sysconv {

typedef __bf16 b2 __attribute__((ext_vector_type(2)));
typedef __bf16 b8 __attribute__((ext_vector_type(8)));
typedef float f2 __attribute__((ext_vector_type(2)));
typedef unsigned u2 __attribute__((ext_vector_type(2)));
typedef unsigned u4 __attribute__((ext_vector_type(4)));

// Three bf16 parts of two numbers; every part is the remainder rounded to nearest.
__device__ __forceinline__ void split2(float a, float b, unsigned& p1, unsigned& p2, unsigned& p3)
{
    p1 = __builtin_bit_cast(unsigned, __builtin_convertvector(f2{a, b}, b2));
    const float ra = a - __builtin_bit_cast(float, p1 << 16), rb = b - __builtin_bit_cast(float, p1 & 0xffff0000u);
    p2 = __builtin_bit_cast(unsigned, __builtin_convertvector(f2{ra, rb}, b2));
    const float sa = ra - __builtin_bit_cast(float, p2 << 16), sb = rb - __builtin_bit_cast(float, p2 & 0xffff0000u);
    p3 = __builtin_bit_cast(unsigned, __builtin_convertvector(f2{sa, sb}, b2));
}

// Inputs below this magnitude (0 apart) are not for the split: with a smallest tap of 2^t, below 2^(-100 - t) products of
// parts that are more than a 2^-26th of the term could fall below 2^-126, and below 2^-103 the parts themselves (below 2^-40 for taps
// down to 2^-60, below 2^-90 for taps from 2^-10 on).  In the form the kernels compare, (bits << 1) - 1, in which +-0 is the largest.
inline unsigned split_tiny_limit(const float* f, int n)
{
    float least = 0x1p40f;
    for (int i = 0; i < n; ++i)
        if (f[i] != 0.0f) least = __builtin_fminf(least, __builtin_fabsf(f[i]));
    int t = 0;
    (void)__builtin_frexpf(least, &t);                                     // least = m 2^t with 1/2 <= m < 1
    const int e = -100 - (t - 1) > -103 ? -100 - (t - 1) : -103;
    return ((unsigned)(127 + e) << 24) - 1u;
}

// Taps the split carries: 0 or 2^-60 .. 2^40 in magnitude, so that no part of a tap and no product of parts is subnormal or
// infinite.  NaN fails too.
inline bool split_takes_taps(const float* f, int n)
{
    for (int i = 0; i < n; ++i) {
        const float a = __builtin_fabsf(f[i]);
        if (!(a == 0.0f || (a >= 0x1p-60f && a <= 0x1p40f))) return false;
    }
    return true;
}

}  // namespace sysconv
