// rewl_replay.h -- repeated additions of ln f to one ln g value in closed form,
// and the margin of a decision on (hi, lo) pairs.
//
// A committed segment adds ln f to a bin once per visit.  Each addition is
// rounded on its own, so the sum is not n ln f; but while the value stays in
// one binade every addition moves it by the same multiple of the spacing U
// there, and n of them are one exact step.  The step is ln f rounded to U, with
// one exception: ln f half-way between two multiples of U rounds to the even
// sum, and its first step depends on the parity of the value.  Such a step
// leaves an even value if it differs from the next one, and steps from an even
// value are all alike; so the step counts as constant once two of them in a row
// are equal.  (Taken at the first value alone, 345 of 2,000,000 replays of the
// pair with ln f = W/t were a spacing off.)
#pragma once

#include "rewl_device.h"

namespace rewl_gpu {

// n >= 1 additions of l to x.  False, and x as it was, where the closed form is
// not known to hold: then they are made one by one.
__host__ __device__ __forceinline__ bool replay_binary64(double &x, double l, uint32_t n) {
#pragma clang fp contract(off)
    // the first addition may enter the binade; the steps behind it stay inside
    const double x1 = x + l, d = (x1 + l) - x1, x2 = x1 + d;
    const double xn = x1 + (double)(n - 1u) * d, z = xn + 4.0 * l;
    const bool binade = ((__builtin_bit_cast(uint64_t, x1) ^ __builtin_bit_cast(uint64_t, z)) >> 52) == 0u;
    if (!(d * 64.0 <= x1 && binade && (x2 + l) - x2 == d)) return false;
    x = xn;
    return true;
}

// Whether x and y are multiples of the binary32 spacing at magnitude m > 0
// (normal range); sums and differences of theirs up to m are then exact.
__host__ __device__ __forceinline__ bool on_grid32(double m, double x, double y) {
#pragma clang fp contract(off)
    int e;
    (void)__builtin_frexp(m, &e);              // m < 2^e: spacing 2^(e - 24)
    const double fx = __builtin_ldexp(x, 24 - e), fy = __builtin_ldexp(y, 24 - e);
    return m > 0x1p-100 && m < 0x1p100 && __builtin_rint(fx) == fx && __builtin_rint(fy) == fy;
}

// n >= 1 additions of l to x, a low word of either sign.  False, and x as it was,
// where the values behind the first leave its binade (or might).
__host__ __device__ __forceinline__ bool replay_low_word(float &x, float l, uint32_t n) {
#pragma clang fp contract(off)
    const float x1 = x + l, x2 = x1 + l, d = x2 - x1;
    const double xn = (double)x1 + (double)(n - 1u) * (double)d;   // exact inside a binade
    const float z = (float)(xn + (double)d);
    const bool binade = ((__builtin_bit_cast(uint32_t, x1) ^ __builtin_bit_cast(uint32_t, z)) >> 23) == 0u;
    if (n > 2u && !(binade && (x2 + l) - x2 == d)) return false;
    x = n == 1u ? x1 : (n == 2u ? x2 : (float)xn);
    return true;
}

// Margin of a decision on the difference d of two pairs, the second with low
// word lo: M and what the binary32 difference may be off.  An infinite ln g of the
// new energy (outside the window, d = -inf) is refused for sure, so d counts up to
// a bound; where ln g of the current energy is infinite, M is.
__host__ __device__ __forceinline__ double pair_margin(double M, double d, float lo) {
#pragma clang fp contract(off)
    return M + (__builtin_fmin(__builtin_fabs(d), 0x1p100) + (double)__builtin_fabsf(lo)) * 0x1p-18;
}

// n additions of l to the pair (hi, lo) by TwoSum.  `any`: whether any lane of
// the wavefront answers yes (for one lane, its own answer).
//
// Single additions cost a turn for all lanes, so closed forms for low words of
// either sign and plain additions for the rest: us per 50,000 attempts on 32 x 32
// sites, 64 walkers, ln f = W/t = 3.9e-7, 4.6e-8 and 4.6e-5: 2223, 1943 and 2967;
// with TwoSum wherever the low word is negative or changes binade 3013, 3088 and
// 3600; with as many steps as the binade holds counted by a division after each
// single addition 3655, 5258 and 7603.
template <class Any>
__host__ __device__ __forceinline__ void replay_pair(float &hi, float &lo, float l, uint32_t n, Any any) {
#pragma clang fp contract(off)
    // where the high word ignores ln f, TwoSum hands it to the low word
    const bool low = hi + l == hi && __builtin_fabsf(hi) < __builtin_inff();
    // n adds that round nowhere, all sums being multiples of the binary32 spacing
    // at the largest of them
    auto exact = [&](float &x) -> bool {
        const double dx = (double)x, dl = (double)l, xn = dx + (double)n * dl;
        if (!on_grid32(__builtin_fmax(__builtin_fabs(dx), __builtin_fabs(xn)), dx, dl)) return false;
        x = (float)xn;
        return true;
    };
    // across binades of the low word only an ln f of few bits does (a power of two)
    const bool few_bits = (__builtin_bit_cast(uint32_t, l) & 0xfffu) == 0u;
    if (n != 0u && low) {
        if ((few_bits && exact(lo)) || replay_low_word(lo, l, n)) n = 0u;
    } else if (n != 0u && exact(hi)) {
        lo = lo + 0.0f;                            // the low word stays (-0 becomes +0, as by TwoSum)
        n = 0u;
    }
    // the others one by one: the low word alone, unless a lane's both words move
    if (any(n != 0u && !low)) {
        while (any(n != 0u)) {
            float xh = hi, xl = lo;
            two_sum_add(xh, xl, l);
            hi = n != 0u ? xh : hi;
            lo = n != 0u ? xl : lo;
            n = n != 0u ? n - 1u : 0u;
        }
    } else {
        while (any(n != 0u)) {
            const float x = lo + l;
            lo = n != 0u ? x : lo;
            n = n != 0u ? n - 1u : 0u;
        }
    }
}

}  // namespace rewl_gpu
