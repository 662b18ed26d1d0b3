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

// How many of n further adds of l to x are known to move it by the constant
// step (x + l) - x: those that stay inside x's binade, counted four short; all
// of them if the step is zero; none if the step after it differs.
__host__ __device__ __forceinline__ uint32_t low_word_steps(float x, float l, uint32_t n) {
#pragma clang fp contract(off)
    const float d = (x + l) - x;
    if (d == 0.0f) return n;
    const float x2 = x + d;
    if (!(x > 0x1p-100f && x < 0x1p100f && d > 0.0f && (x2 + l) - x2 == d)) return 0u;
    int e;
    (void)__builtin_frexpf(x, &e);             // x < 2^e
    const float room = (__builtin_ldexpf(1.0f, e) - x) / d - 4.0f;
    const uint32_t k = room >= 64.0f ? 64u : (room >= 1.0f ? (uint32_t)room : 0u);
    return k < n ? k : n;
}

// Margin of a decision on the difference d of two pairs, the second with low
// word lo: M and what the binary32 difference may be off.  An infinite ln g of the
// new energy (outside the window, d = -inf) is refused for sure, so d counts up to
// a bound; where ln g of the current energy is infinite, M is.
__host__ __device__ __forceinline__ double pair_margin(double M, double d, float lo) {
#pragma clang fp contract(off)
    return M + (__builtin_fmin(__builtin_fabs(d), 0x1p100) + (double)__builtin_fabsf(lo)) * 0x1p-18;
}

// n additions of l to the pair (hi, lo) by TwoSum.  `any` says whether the loop
// over single additions goes on, given that this lane still has some (on the
// GPU for all lanes of a wavefront together).
template <class Any>
__host__ __device__ __forceinline__ void replay_pair(float &hi, float &lo, float l, uint32_t n, Any any) {
#pragma clang fp contract(off)
    // n adds that round nowhere, all sums being multiples of the
    // binary32 spacing at the largest of them: in the high word
    // the low word then stays; where the high word ignores ln f
    // TwoSum hands it to the low word, which takes them all
    const bool low = hi + l == hi;
    if (n != 0u) {
        const double dl = (double)l, sh = (double)hi + (double)n * dl, sl = (double)lo + (double)n * dl;
        if (on_grid32(__builtin_fmax(__builtin_fabs((double)hi), __builtin_fabs(sh)), (double)hi, dl)) {
            hi = (float)sh;
            lo = lo + 0.0f;                        // (-0 becomes +0, as by TwoSum)
            n = 0u;
        } else if (low && on_grid32(__builtin_fmax(__builtin_fabs((double)lo), __builtin_fabs(sl)), (double)lo, dl)) {
            lo = (float)sl;
            n = 0u;
        }
    }
    // otherwise one add, then in the low word as many of its
    // constant steps (see above) as its binade holds
    while (any(n != 0u)) {
        float xh = hi, xl = lo;
        two_sum_add(xh, xl, l);
        hi = n != 0u ? xh : hi;
        lo = n != 0u ? xl : lo;
        n = n != 0u ? n - 1u : 0u;
        const uint32_t skip = low ? low_word_steps(lo, l, n) : 0u;
        lo = skip != 0u ? (float)((double)lo + (double)skip * (double)((lo + l) - lo)) : lo;
        n -= skip;
    }
}

}  // namespace rewl_gpu
