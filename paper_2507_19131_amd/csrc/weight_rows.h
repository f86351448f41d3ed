// What a block's creation takes from the rows of its weight codes, and which integer sums over them stay small.  Host code.
#pragma once
#include <stdint.h>
#include <algorithm>

namespace mixaq {

struct RowCodes { int sum, width, lowest, highest; };               // of w, of |w|, and the extreme codes
// Two plain loops, which become vector instructions (7.1 million weights of a block of C = 768: one loop that also leaves at the first code
// out of range 12.6 ms, these 2.0).
inline RowCodes row_codes(const int8_t* w, int K)
{
    int sum = 0, width = 0;
    for (int k = 0; k < K; ++k) {
        sum += w[k];
        width += w[k] < 0 ? -w[k] : w[k];
    }
    uint8_t low = 255, high = 0;                                     // of code + 128
    for (int k = 0; k < K; ++k) {
        const uint8_t u = (uint8_t)(w[k] ^ -128);
        low = std::min(low, u);
        high = std::max(high, u);
    }
    return {sum, width, low - 128, high - 128};
}

// Whether every sum over k of (code - zp) W[n,k], codes in [qmin, qmax] and rows of at most `width` in absolute value, lies inside +-2^22,
// where a binary32 of magnitude 1.5 * 2^23 holds it as its own bits.
constexpr int SUM_MAGIC_BOUND = 1 << 22;
inline bool sums_fit(int width, int qmin, int qmax, int zp) { return (long long)width * std::max(qmax - zp, zp - qmin) < SUM_MAGIC_BOUND; }

}  // namespace mixaq
