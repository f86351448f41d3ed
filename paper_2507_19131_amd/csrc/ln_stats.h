// LayerNorm statistics of one token, binary64: the sum first, then the squares centred on the ROUNDED mean, each rounded to
// binary32 once.  Plain arithmetic without GPU builtins, so that the same lines are compiled for the host and compared there
// with exact arithmetic (tests/test_layernorm_statistics.py).
//
// Two passes over the registers of a token (convert and add, then convert, subtract and fused multiply-add: five vector
// instructions per element).  Sum and sum of squares in one pass take three, but sum (x - mean)^2 = q - mean (2 s - C mean)
// cancels: its relative error grows with 1 + mean^2 / var, 60 times this one's at mean = 7 standard deviations, and is above it
// at every ratio.
#pragma once
#include <math.h>

#if defined(__HIPCC__)
#define MIXAQ_HD __host__ __device__ __forceinline__
#else
#define MIXAQ_HD static inline
#endif

namespace mixaq {

MIXAQ_HD double sum4(float a, float b, float c, float d) { return ((double)a + (double)b) + ((double)c + (double)d); }

// REREAD: the caller's four registers are made opaque (in place: a copy costs a move per element), or the compiler keeps their conversions to binary64 from the first pass in registers,
// twice the token, in spills where the registers are full (the window kernel's forms of a pair of waves per head: up to 58).  The
// token kernel and the 96-channel embedding have the room: a conversion less per element, 4 x 128 x 128 x 256 333.5 -> 330.6 us the
// pair of blocks, 4 x 256 x 256 x 128 448.5 -> 446.0, embedding 800 x 1344 on fresh images 13.25 -> 13.05.
template <bool REREAD, class F>
MIXAQ_HD double centred4(F& x0, F& x1, F& x2, F& x3, float mean)
{
#if defined(__HIP_DEVICE_COMPILE__)
    if (REREAD) asm("" : "+v"(x0), "+v"(x1), "+v"(x2), "+v"(x3));
#endif
    const double m = mean, a = (double)x0 - m, b = (double)x1 - m, c = (double)x2 - m, d = (double)x3 - m;
    return __builtin_fma(a, a, b * b) + __builtin_fma(c, c, d * d);
}

// v / C for the widths of the blocks and mergings, C = 2^k or 3 * 2^k: the bits of the division in three instructions.  1 / C
// rounded is exact or low by 2^-54 of itself, so q is within one unit of its last place of v / C, the residual is exact, and
// one correction step rounds correctly (Markstein 1990).
MIXAQ_HD double over_channels(double v, int C)
{
    const double c = C, r = 1.0 / c, q = v * r;
    return __builtin_fma(__builtin_fma(-q, c, v), r, q);
}
MIXAQ_HD float ln_mean(double sum, int C) { return (float)over_channels(sum, C); }
MIXAQ_HD float ln_var(double centred, int C) { return (float)over_channels(centred, C); }
MIXAQ_HD float ln_rstd(double centred, int C, float eps) { return 1.0f / sqrtf(ln_var(centred, C) + eps); }

}  // namespace mixaq
