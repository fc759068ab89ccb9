// near_log.h -- the logarithm of the FP64 logarithmic near field (p2p.hip).  Plain
// C++ as well, so that its arithmetic is tested value by value on the CPU
// (tests/test_near_log.py).
#pragma once

#include <cmath>
#include <cstdint>

#ifdef __HIP__
#define FMM_LOG_FN __host__ __device__ __forceinline__
#else
#define FMM_LOG_FN inline
#endif

namespace fmm {

constexpr int kLogTab = 128;
// log(2) / 2 in two parts: the first a multiple of 2^-43 (its product with an
// exponent is exact), the second the rest
constexpr double kHalfLn2Hi = 0x1.62e42fefa38p-2, kHalfLn2Lo = 0x1.ef35793c7673p-46;

// The table: interval t of the top seven bits of the mantissa of x, half an exponent
// up (t >= 64: m in [1 + (t-64)/128, + 1/128), t < 64: m in [3/4 + t/256, + 1/256)).
// 1/c is 1/m at its middle rounded to a multiple of 2^-7 below m = 1 and of 2^-8
// above it, 1 for the two intervals next to m = 1.  An entry is log(c)/2 in two
// parts: x a multiple of 2^-43, y the rest, of which the low 32 bits are replaced by
// those of 1/(2c) as a float (they weigh less than 2^-65), xor kOneHalf so that
// both parts are exactly zero for c = 1.
constexpr uint32_t kOneHalf = 0x3f000000u;
template <class D2>
void log_table(D2* tab)
{
    for (int t = 0; t < kLogTab; ++t) {
        const bool one = t == kLogTab / 2 - 1 || t == kLogTab / 2;    // next to m = 1
        const long double mid = t >= kLogTab / 2 ? 1.0L + (t - kLogTab / 2 + 0.5L) / 128 : 0.75L + (t + 0.5L) / 256;
        const long double grid = t >= kLogTab / 2 ? 256.0L : 128.0L;
        const long double inv = one ? 1.0L : std::rint(grid / mid) / grid;
        const long double h = one ? 0.0L : -std::log(inv) / 2;
        const double hi = (double)(std::rint(h * 0x1p43L) * 0x1p-43L);
        const uint64_t half_inv = __builtin_bit_cast(uint32_t, (float)(inv / 2)) ^ kOneHalf;
        const long double lo = h - hi;
        double best = 0.0;
        const int64_t top = (int64_t)(__builtin_bit_cast(uint64_t, (double)lo) >> 32);
        for (int64_t k = top > 0 ? top - 1 : 0; k <= top + 1; ++k) {
            const double y = __builtin_bit_cast(double, (uint64_t)k << 32 | half_inv);
            if (k == (top > 0 ? top - 1 : 0) || std::fabs(y - lo) < std::fabs(best - lo)) best = y;
        }
        tab[t].x = hi;
        tab[t].y = best;
    }
}

// log(x) / 2 of a positive normal number: x = 2^e m with m in [3/4, 3/2), 1/c from
// the table, r = m / c - 1 (exact: |r| <= 2^-7 and a multiple of 2^-60), log x =
// e log 2 + log c + log(1 + r), everything halved (Tang's table-driven method: the
// sum of the leading parts and r with its rounding error, to which the parts'
// rests and the series are added).  The series is Taylor's to r^8, its last term
// economised (Chebyshev; 2^-57 of the result at most).  Largest error found 0.556
// units in the last place of the result, rms 0.289 (the device library's
// logarithm: 0.638, 0.296; with log 2 and log c in one part each and nothing
// compensated: 1.67, 0.47).  fmm_evaluate_log at N = 5e5, 8 levels, FP64, p = 16: 398
// us, with the library's logarithm 797 us, uncompensated 371 us.
template <class D2>
FMM_LOG_FN double half_log(double x, const D2* tab)
{
    const uint64_t u = __builtin_bit_cast(uint64_t, x);
    const int hi = (int)(u >> 32), t = hi + 0x00080000;   // half: the exponent of m >= 3/2 moves up
    const int ne = 1023 - (t >> 20);                       // -e
    const D2 c = tab[(t >> 13) & (kLogTab - 1)];
    const double half_inv =
        (double)__builtin_bit_cast(float, (uint32_t)__builtin_bit_cast(uint64_t, (double)c.y) ^ kOneHalf);
    const double m = __builtin_bit_cast(double, (uint64_t)(uint32_t)(hi + (ne << 20)) << 32 | (uint32_t)u);
    const double r = fma(m, half_inv, -0.5), e = (double)ne;
    const double w = fma(e, -kHalfLn2Hi, c.x);             // exact
    const double s = w + r;
    const double rest = ((w - s) + r) + fma(e, -kHalfLn2Lo, c.y);
    double p = fma(r, 64.0 / 7, -16.0 / 3 - 24 * 0x1p-16);
    p = fma(r, p, 16.0 / 5);
    p = fma(r, p, -2.0 + 9 * 0x1p-32);
    p = fma(r, p, 4.0 / 3);
    p = fma(r, p, -1.0 - 0x1p-49);
    const double v = s + fma(r * r, p, rest);
    return hi < 0x7ff00000 ? v : x;                        // x overflowed: infinite
}

}  // namespace fmm
