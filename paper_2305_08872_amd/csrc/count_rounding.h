// The fp32 count's predicate in two operations that need neither the rounded product nor its comparison:
//
//     t   = clamp(fma(a, b g, -th g), 0, 1)       g = 1 / (distance from th to the next float above)
//     sum = fma(t, s, sum)                        sum in [2^23, 2^24), where it has no fraction
//
// and sum - 2^23 is the number of products with RN(a b) > th.  Why this is exact:
//   * g is a power of two, so b g is b with another exponent and th g is a whole number of at most 24 bits;
//     the first fma's t is (a b - th) in units of that distance.
//   * RN(a b) > th exactly when a b lies more than half the distance above th, or half of it and th is odd (its
//     last bit is set: the tie goes to the even neighbour above).  So the predicate is t against 1/2.
//   * a b is a product of two numbers of 24 bits, and for 0 < t < 1 it lies between th and its neighbour: it is a multiple
//     of 2^-47 of its power of two, t of 2^-24, which fp32 holds exactly from 1/4 on.
//   * the second fma rounds sum + t s to a whole number, once.  With s = 1 - 2^-24 (th even) t = 1/2 rounds down and
//     1/2 + 2^-24, the next one, up; with s = 1 + 2^-23 (th odd) t = 1/2 rounds up and 1/2 - 2^-24 down; 0 and 1
//     add 0 and 1.
// Below a negative power of two the next float is half as far as below its neighbours: g is taken from there.
// (NaN products: the clamp makes them 0, as not above.  An infinite threshold has g = 1.)
//
// It holds for thresholds of magnitudes 2^-40 to 2^24 (g >= 1: no b g loses bits) as long as no b g overflows, which the
// kernels watch (b would have to be 2^105 times the threshold).  Tiles with other thresholds -- smaller, larger, NaN, zeros beside
// others -- take the comparison.
//
// Where all thresholds of a tile are zero, RN(a b) > 0 is counted, a b > 2^-150 (2^-150 itself ties to zero), by the same two operations:
//     t = clamp(fma(a', b', -2^47)),  a' b' = 2^197 a b,  s = 1
// a b 2^150 is a multiple of 2^-47 around 1, so t is 1 above it, and 0 at it and below.  The tile kernels put 2^98 on A and 2^99 on B
// as they are read from LDS; what overflows there is as good infinite: times a nonzero factor t is 1 or 0, and times zero NaN, t 0.
// In the wide kernel, whose A stays in scalar registers, both factors go on B as it is staged, one after the other.  b' then
// overflows from 2^-69 on, and a nonzero |a| below 2^-80 could make a product that rounds to zero: the rows of A are read once
// ahead of the loop, and such a value sends the tile to the comparison.
//
// Bound: vector-ALU issue, 4.7 clocks per 64 products in a register-only loop (a in a scalar register) where multiply, subtract and the
// sign bit shifted in take 6.5.  The wide kernel, us, by comparison / so / thresholds of zero: 4096^3 3110 / 2420 / 2380, thresholds that face
// rows 3030 / 2750 / 2255, one 3030 / 2340 / 2240, A transposed 3820 / 2960, B transposed 3150 / 2420 / 2250; 2048^3 398 / 308 / 316, 1536^3 191 (in
// the tile kernels) / 150 / 162.  Not for thresholds per output (a factor each).  The tile kernels, which read both operands from LDS and
// are bound there too, gain 4 to 18 % from 15 us on, with thresholds of zero too (mmlike_tile_impl.h).
#include <hip/hip_runtime.h>
#include <stdint.h>

#ifndef AMULET_COUNT_ROUNDING_H
#define AMULET_COUNT_ROUNDING_H

namespace amulet {

constexpr float COUNT_ROUNDING_ZERO = 0x1p23f;
constexpr float COUNT_ZERO_A = 0x1p98f, COUNT_ZERO_B = 0x1p99f, COUNT_ZERO_NEG = -0x1p47f;
constexpr uint32_t COUNT_ZERO_LEAST = ((127u - 80u) << 24) - 1u;     // twice the bits of 2^-80, less 1 (a zero's are the largest)
constexpr int COUNT_ROUNDING_K = (1 << 23) - 1;      // products a sum holds

// g, s and -th g of a threshold; whether it has them
__device__ __forceinline__ bool count_rounding(float th, float &g, float &s, float &neg)
{
    const uint32_t bits = __builtin_bit_cast(uint32_t, th);
    const int exponent = (int)((bits >> 23) & 255) - 127;
    const int e = exponent - ((bits & 0x807fffffu) == 0x80000000u ? 1 : 0);
    const bool inf = (bits & 0x7fffffffu) == 0x7f800000u, in_range = exponent >= -40 && exponent < 24;
    g = in_range ? __builtin_bit_cast(float, (uint32_t)(150 - e) << 23) : 1.0f;
    s = (bits & 1u) ? 0x1.000002p0f : 0x1.fffffep-1f;
    neg = -th * g;
    return inf || in_range;
}

// four products of a with b, one of which carries g
__device__ __forceinline__ void count_by_rounding4(float a, const float *b, const float *neg, const float *s, float *sum)
{
    float t[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) t[c] = __builtin_amdgcn_fmed3f(__builtin_fmaf(a, b[c], neg[c]), 0.0f, 1.0f);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int c = 0; c < 4; ++c) sum[c] = __builtin_fmaf(t[c], s[c], sum[c]);
}

}  // namespace amulet
#endif
