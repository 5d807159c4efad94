// The tile form's rows on the matrix cores: operands of one
// v_mfma_f32_32x32x16_bf16 from floats split into bfloat16 pieces (Henry, Tang and
// Heinecke, ARITH 2019), and the bound on the error of the decisions made from its
// results.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace hg {

// Where a pair's points lie (those with four finite coordinates; the others are
// outliers to every hypothesis): x1 and y1 within r1 of c1, and x2 / tau and
// y2 / tau, in the float arithmetic of the scoring, within r2 of k2.
struct Extent {
  float c1[2], k2[2], r1[2], r2[2];
};

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Two floats rounded to nearest bfloat16 (a in the low half).
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  const bf16x2 v = {static_cast<__bf16>(a), static_cast<__bf16>(b)};
  return __builtin_bit_cast(uint32_t, v);
}
__device__ __forceinline__ float high_bf16(uint32_t p) {
  return __uint_as_float(p & 0xffff0000u);
}

// Operand B of a point: this lane's coordinate c (x1 or y1); one = its
// constants (1 1 or 1 0).
__device__ __forceinline__ bf16x8 point_operand(float c, uint32_t one) {
  u32x4 v;
  v[0] = pack_bf16(c, c);
  const float r1 = c - high_bf16(v[0]);
  v[1] = pack_bf16(r1, r1);
  const float r2 = r1 - high_bf16(v[1]);
  v[2] = pack_bf16(c, r2);
  v[3] = one;
  return __builtin_bit_cast(bf16x8, v);
}

// The three bfloat16 pieces of a float, as floats (their sum is exactly x).
__device__ __forceinline__ void pieces(float x, float f[3]) {
  f[0] = x;
  f[1] = x - high_bf16(pack_bf16(0.0f, x));
  f[2] = f[1] - high_bf16(pack_bf16(0.0f, f[1]));
}

// Operand A of one row, the slots of one half: g = its x1 or y1 coefficient, c =
// its constant (rounded by pack_bf16, which leaves the pieces).
__device__ __forceinline__ u32x4 row_operand(const float g[3], const float c[3], int half) {
  u32x4 v;
  v[0] = v[1] = pack_bf16(g[0], g[1]);
  v[2] = pack_bf16(g[2], g[0]);
  v[3] = half ? pack_bf16(c[2], 0.0f) : pack_bf16(c[0], c[1]);
  return v;
}

// Bound on |e_computed - e| for the tile form over points with |x1 - c| <=
// r1[0], |y1 - c| <= r1[1], |x2c| <= r2[0], |y2c| <= r2[1], rows g on centred
// coordinates; e = ru^2 + rv^2 - w^2. With u = 2^-24, SU = |g0| r1[0] + |g1| r1[1] +
// |g2| and SV, SW likewise for rows 2 and 3:
//  * The matrix instruction takes slots 0 - 7, then 8 - 15. It cuts each of the 8
//    products to a multiple of 2^-24 of their largest power of two (the sum of two
//    operands' exponents), adds them exactly, and adds that sum, cut at 2^-31, to the
//    sum so far, cut at 2^-24, of the larger power of the two, and rounds to float. (Found
//    by experiment, and held bit for bit over random, wide-range and cancelling rows
//    by tests/test_gpu_tile_rows.py.) The largest product is not cut, so a step
//    loses at most 7 u of its own products' magnitude sum, the cut of the first
//    step's sum u of the second's products, and each rounding u of the sum: 9.01 u of
//    all products' magnitude sum, which is at most 1.016 of the row's.
//  * The three products of pieces that are left out are at most 2.01 u of the row's
//    magnitude sum: a row of floats errs by at most kRowError = 11.25 u of it.
//  * The rounding of g to float and of the centred point add 1 u each: 13.25 u of
//    SU, SV or SW. With the rounding of x2c and y2c (1 u), ru and rv err together by
//    S = 14.5 u (SU + SV + (r2[0] + r2[1]) SW) beside their own rounding.
//  * A wrong decision needs the true or the computed d = ru^2 + rv^2 at or below
//    w^2 <= SW^2, so that |(ru, rv)| <= SW (1 + small). Then e errs by 2 SW S + S^2
//    from the residuals, 26.5 u SW^2 (and a square) from w, 2 u d from 1/tau, which
//    enters squared, and 4 u d from the residuals' roundings, the squares and sums:
//    2 SW S + S^2 + 32.5 u SW^2, which is below
//      SW (36 u SW + 2.25 S) + 2 S^2
//    by a tenth, for sigma's rounding, for sums that agree by rounding and for the
//    float64 test's own error.
// The row errors that occur are smaller: at most 4.3 u, 0.8 u rms over the test's two
// million rows (float FMAs of the same entries: 1.9 u, 0.5 u rms). They decide how
// many points stay open, not how any is counted: the bound costs 1 % of a call
// (512 pairs of up to 8000 points x 1024: 541 us with the smaller bound that the
// errors seen would allow, 546 us).
// False: the magnitudes leave the range where that holds (the hypothesis is
// then counted in float64 throughout). Of it: a coordinate past 3.38e38 rounds to an
// infinite piece, and pieces below 2^-133 are lost. With coordinates below 1e18 and
// scaled entries below 1e25 (kMaxEntry) the latter move a row by less than 1e-12,
// and e, scaled, by less than 1e-6 of its bound.
constexpr float kRowError = 11.25f;   // in units of 2^-24 of the magnitude sum
constexpr double kMaxEntry = 1.0e25;
__device__ __forceinline__ bool tile_bound(const double *g, const Extent &x, float &bound) {
  constexpr float u = 5.9604645e-08f;   // 2^-24
  float s[3];
#pragma unroll
  for (int r = 0; r < 3; ++r)
    s[r] = fmaf(fabsf(static_cast<float>(g[3 * r])), x.r1[0],
                fmaf(fabsf(static_cast<float>(g[3 * r + 1])), x.r1[1],
                     fabsf(static_cast<float>(g[3 * r + 2]))));
  const float sw = s[2];
  const float mag = fmaf(x.r2[0] + x.r2[1], sw, s[0] + s[1]);
  const float S = (14.5f * u) * mag;
  bound = fmaf(sw, fmaf(36.0f * u, sw, 2.25f * S), fmaf(2.0f * S, S, 1.0e-35f));
  return mag + sw < 1.0e18f && sw > 1.0e-18f && fmaxf(x.r1[0], x.r1[1]) < 1.0e18f;
}

}  // namespace hg
