// Batched 4-point solver: one quadruple per lane. Each wave reads 256
// contiguous bytes from each of the 16 input planes and writes 256 bytes to
// each of the 9 output planes (plus 64 flag bytes): memory-bound at 101 B per
// quadruple, with the double-precision arithmetic hidden under the HBM time.
// Measured on MI355X, this shape (512-thread workgroups, one quadruple per
// lane, a grid that covers the batch once) streams faster than four quadruples
// per lane with 16-byte accesses, except near n = 2^20, where all of their
// workgroups are resident at once (25 us to 22; n = 3.2e6: 56 us to 66).
//
// Loads and stores are non-temporal while a wave's 256 bytes of a plane are
// whole lines (STREAM). Where they are not, two waves share the line between
// them, and a non-temporal access gives the line up after the first: it is
// fetched twice, and written to memory as two partial lines. Ordinary accesses
// let the second wave find it in L2, which joins the two writes. SKS solver,
// planes n floats apart, non-temporal and ordinary: n = 512003, 15.2 and 14.1
// us; 1024003, 27.8 and 25.6; 3200003, 74.8 and 65.1; 12800003, 302 and 247
// (simplified SK 11.3 and 9.2, 19.5 and 19.3, 54.4 and 47.1, 217 and 174);
// where the lines are whole the non-temporal accesses win (n = 3200000, 56.2
// and 61.4; 12800000, 217 and 232).
#include <cmath>

#include "common.hpp"
#include "solver_dev.hpp"

namespace hg {

constexpr int kSolveThreads = 512;

template <bool STREAM, typename T>
__device__ __forceinline__ T plane_load(const T *p) {
  return STREAM ? __builtin_nontemporal_load(p) : *p;
}

template <bool STREAM, typename T>
__device__ __forceinline__ void plane_store(T v, T *p) {
  if (STREAM)
    __builtin_nontemporal_store(v, p);
  else
    *p = v;
}

// Whether every float plane starts on a 64-byte sector: one half of a line off
// costs less than the ordinary accesses would (planes 64 k + 16 floats apart,
// n = 1000003: 22.0 us against 22.7; simplified SK 15.5 against 16.5), a
// quarter costs more at large n (64 k + 8, n = 4194309: 104 against 94.9; 73.2
// against 69.0). A batch below kSharedLinesMin stays in the caches either way,
// and the two differ by less than their own spread (n = 256003: 7.3 and 7.6 us).
constexpr int64_t kSharedLinesMin = 1 << 18;
static bool stream_planes(const void *a, const void *b, const void *c, int64_t n, int64_t ld) {
  const uintptr_t bits = reinterpret_cast<uintptr_t>(a) | reinterpret_cast<uintptr_t>(b) |
                         reinterpret_cast<uintptr_t>(c) | static_cast<uintptr_t>(4 * ld);
  return (bits & 63) == 0 || n <= kSharedLinesMin;
}

// Order of the workgroups over the batch. Consecutive workgroups go to the 8 XCDs
// in turn, so in linear order every XCD touches every 16 KB of every plane. Grouped
// order gives an XCD 2^log_group consecutive workgroups of every 8 times as many.
// It is taken where the planes' starts fall together:
//  * on planes that do not start on lines, where neighbours share them and an XCD's
//    L2 then holds both sides; 32 workgroups (SKS solver, linear and grouped:
//    n = 1000003, 23.7 and 22.9 us; 4194309, 98.3 and 88.1; 12800003, 247 and 242;
//    simplified SK 18.1 and 17.5, 73.8 and 64.4, 171 and 163);
//  * on planes a multiple of 4 MB apart up to 2^23 problems, whose accesses meet in
//    the same memory channels; 256 workgroups (512 KB of each plane) between 2^20
//    and 2^23, 32 at these ends (linear, 32 and 256; 2^20: 24.6, 22.0, 23.8; 2^21:
//    44.6, 40.7, 38.2; 2^22: 86.4, 80.9, 71.4; 6 2^20: 116, 112, 108; simplified SK
//    17.3, 15.8, 17.9; 32.4, 28.5, 26.7; 62.6, 57.9, 49.3; 85.2, 75.1, 71.8; 2^23:
//    109 - 118, 98.2, 102).
// Elsewhere linear order streams better (linear and 32: n = 3200000, 56.4 and 57.1;
// 2^24, 278 and 286; simplified SK 39.1 and 39.7, 188 and 193).
constexpr uint32_t kXcds = 8;
struct BlockOrder {
  uint32_t grouped;     // the workgroups that are permuted, in runs of kXcds 2^log_group
  uint32_t log_group;
};
static BlockOrder block_order(bool stream, int64_t n, int64_t ld, unsigned grid) {
  const bool same_channels = ld % (1 << 20) == 0 && n > kSharedLinesMin && n <= (1 << 23);
  if (stream && !same_channels) return {0u, 0u};
  const uint32_t lg = stream && n > (1 << 20) && n < (1 << 23) ? 8u : 5u;
  return {grid >> lg >> 3 << lg << 3, lg};
}

// The first problem of a thread.
__device__ __forceinline__ int64_t first_problem(const BlockOrder &o) {
  const uint32_t b = blockIdx.x, in = b & ((kXcds << o.log_group) - 1u);
  const uint32_t tile = b < o.grouped ? b - in + (in % kXcds << o.log_group) + in / kXcds : b;
  return static_cast<int64_t>(tile) * kSolveThreads + threadIdx.x;
}

template <int METHOD, bool STREAM>
__global__ __launch_bounds__(kSolveThreads) void solve4_kernel(const float *__restrict__ src,
                                                               const float *__restrict__ dst,
                                                               int64_t n, int64_t ld,
                                                               BlockOrder order,
                                                               float *__restrict__ H,
                                                               uint8_t *__restrict__ flags) {
  const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
  for (int64_t q = first_problem(order); q < n; q += stride) {
    float s[8], d[8], h[9];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      s[k] = plane_load<STREAM>(src + k * ld + q);
      d[k] = plane_load<STREAM>(dst + k * ld + q);
    }
    const uint32_t f = solve_quad<METHOD>(s, d, h);
#pragma unroll
    for (int k = 0; k < 9; ++k) plane_store<STREAM>(h[k], H + k * ld + q);
    if (flags) plane_store<STREAM>(static_cast<uint8_t>(f), flags + q);
  }
}

template <int METHOD, bool STREAM>
static int launch_solve(const float *src, const float *dst, int64_t n, int64_t ld, float *H,
                        uint8_t *flags, hipStream_t s) {
  // one pass over the batch; beyond 2^31 - 1 workgroups the grid-stride loop takes over
  const int64_t blocks = (n + kSolveThreads - 1) / kSolveThreads;
  const unsigned grid = static_cast<unsigned>(blocks > 0x7FFFFFFF ? 0x7FFFFFFF : blocks);
  hipLaunchKernelGGL((solve4_kernel<METHOD, STREAM>), dim3(grid), dim3(kSolveThreads), 0, s, src, dst, n,
                     ld, block_order(STREAM, n, ld, grid), H, flags);
  return launched("solve4_kernel");
}

// Simplified SK over n images of one pattern: 8 target planes in, 9 planes of
// Hbar and the flags out (69 B per problem).
template <bool STREAM>
__global__ __launch_bounds__(kSolveThreads) void sk_kernel(SkPattern pat,
                                                           const float *__restrict__ dst,
                                                           int64_t n, int64_t ld, BlockOrder order,
                                                           float *__restrict__ H,
                                                           uint8_t *__restrict__ flags) {
  const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
  for (int64_t q = first_problem(order); q < n; q += stride) {
    float d[8], h[9];
#pragma unroll
    for (int k = 0; k < 8; ++k) d[k] = plane_load<STREAM>(dst + k * ld + q);
    const uint32_t f = solve_sk(pat, d, h);
#pragma unroll
    for (int k = 0; k < 9; ++k) plane_store<STREAM>(h[k], H + k * ld + q);
    if (flags) plane_store<STREAM>(static_cast<uint8_t>(f), flags + q);
  }
}

// Three-point affine: 6 + 6 planes in, 6 planes of A and the flags out
// (73 B per problem).
template <bool STREAM>
__global__ __launch_bounds__(kSolveThreads) void affine_kernel(const float *__restrict__ src,
                                                               const float *__restrict__ dst,
                                                               int64_t n, int64_t ld, BlockOrder order,
                                                               float *__restrict__ A,
                                                               uint8_t *__restrict__ flags) {
  const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
  for (int64_t q = first_problem(order); q < n; q += stride) {
    float s[6], d[6], a[6];
#pragma unroll
    for (int k = 0; k < 6; ++k) {
      s[k] = plane_load<STREAM>(src + k * ld + q);
      d[k] = plane_load<STREAM>(dst + k * ld + q);
    }
    const uint32_t f = solve_affine(s, d, a);
#pragma unroll
    for (int k = 0; k < 6; ++k) plane_store<STREAM>(a[k], A + k * ld + q);
    if (flags) plane_store<STREAM>(static_cast<uint8_t>(f), flags + q);
  }
}

static unsigned one_pass_grid(int64_t n) {
  const int64_t blocks = (n + kSolveThreads - 1) / kSolveThreads;
  return static_cast<unsigned>(blocks > 0x7FFFFFFF ? 0x7FFFFFFF : blocks);
}

// Per-pattern constants of the simplified SK, in the operation order of the
// per-image steps (double precision on the host, once per call).
static SkPattern sk_pattern(const double *o, double *frame) {
  const double ONx = (o[2] - o[0]) * 0.5, ONy = (o[3] - o[1]) * 0.5;
  const double Ox = o[0] + ONx, Oy = o[1] + ONy;
  const double f = ONx * ONx + ONy * ONy;
  double dx = o[4] - Ox, dy = o[5] - Oy;
  const double P3x = ONx * dx + ONy * dy, P3y = ONx * dy - ONy * dx;
  double r = 1.0 / P3y;
  SkPattern p;
  p.P5x = P3x * r;
  p.P5y = f * r;
  dx = o[6] - Ox;
  dy = o[7] - Oy;
  const double Q3x = ONx * dx + ONy * dy, Q3y = ONx * dy - ONy * dx;
  r = 1.0 / Q3y;
  const double Q7x = Q3x * r - p.P5x, Q7y = f * r - p.P5y;
  p.kp = 1.0 / (Q7x + Q7y);
  p.km = 1.0 / (Q7x - Q7y);
  p.flags = quad_side_thin(o) ? kNearDegenerate : 0u;
  if (frame) {  // H_S1 of eq. 3_2_4
    const double tx = -(ONx * Ox + ONy * Oy), ty = ONy * Ox - ONx * Oy;
    const double m[9] = {ONx, ONy, tx, -ONy, ONx, ty, 0.0, 0.0, f};
    for (int i = 0; i < 9; ++i) frame[i] = m[i];
  }
  return p;
}

}  // namespace hg

extern "C" int hg_solve4(int method, const float *src, const float *dst, int64_t n, int64_t ld,
                         float *H, uint8_t *flags, void *stream) {
  hg::clear_error();
  HG_REQUIRE(method == HG_ACA || method == HG_SKS, "hg_solve4: unknown method %d", method);
  HG_REQUIRE(n >= 0, "hg_solve4: n = %lld < 0", static_cast<long long>(n));
  if (n == 0) return HG_OK;
  HG_REQUIRE(src && dst && H, "hg_solve4: NULL src, dst or H");
  HG_REQUIRE(ld >= n, "hg_solve4: ld = %lld < n = %lld", static_cast<long long>(ld),
             static_cast<long long>(n));
  HG_REQUIRE(ld <= (INT64_MAX / 16), "hg_solve4: ld too large");
  const hipStream_t s = hg::as_stream(stream);
  const auto launch = hg::stream_planes(src, dst, H, n, ld)
                          ? (method == HG_ACA ? hg::launch_solve<0, true> : hg::launch_solve<1, true>)
                          : (method == HG_ACA ? hg::launch_solve<0, false>
                                              : hg::launch_solve<1, false>);
  return launch(src, dst, n, ld, H, flags, s);
}

extern "C" int hg_solve_sk(const double *obj, const float *dst, int64_t n, int64_t ld, float *H,
                           uint8_t *flags, double *frame, void *stream) {
  hg::clear_error();
  HG_REQUIRE(obj, "hg_solve_sk: NULL pattern");
  for (int k = 0; k < 8; ++k)
    HG_REQUIRE(std::isfinite(obj[k]), "hg_solve_sk: pattern coordinate %d is not finite", k);
  HG_REQUIRE(n >= 0, "hg_solve_sk: n = %lld < 0", static_cast<long long>(n));
  const hg::SkPattern pat = hg::sk_pattern(obj, frame);
  if (n == 0) return HG_OK;
  HG_REQUIRE(dst && H, "hg_solve_sk: NULL dst or H");
  HG_REQUIRE(ld >= n, "hg_solve_sk: ld = %lld < n = %lld", static_cast<long long>(ld),
             static_cast<long long>(n));
  HG_REQUIRE(ld <= (INT64_MAX / 16), "hg_solve_sk: ld too large");
  const bool nt = hg::stream_planes(dst, H, H, n, ld);
  const unsigned grid = hg::one_pass_grid(n);
  hipLaunchKernelGGL((nt ? hg::sk_kernel<true> : hg::sk_kernel<false>), dim3(grid),
                     dim3(hg::kSolveThreads), 0, hg::as_stream(stream), pat, dst, n, ld,
                     hg::block_order(nt, n, ld, grid), H, flags);
  return hg::launched("sk_kernel");
}

extern "C" int hg_solve3_affine(const float *src, const float *dst, int64_t n, int64_t ld,
                                float *A, uint8_t *flags, void *stream) {
  hg::clear_error();
  HG_REQUIRE(n >= 0, "hg_solve3_affine: n = %lld < 0", static_cast<long long>(n));
  if (n == 0) return HG_OK;
  HG_REQUIRE(src && dst && A, "hg_solve3_affine: NULL src, dst or A");
  HG_REQUIRE(ld >= n, "hg_solve3_affine: ld = %lld < n = %lld", static_cast<long long>(ld),
             static_cast<long long>(n));
  HG_REQUIRE(ld <= (INT64_MAX / 16), "hg_solve3_affine: ld too large");
  const bool nt = hg::stream_planes(src, dst, A, n, ld);
  const unsigned grid = hg::one_pass_grid(n);
  hipLaunchKernelGGL((nt ? hg::affine_kernel<true> : hg::affine_kernel<false>), dim3(grid),
                     dim3(hg::kSolveThreads), 0, hg::as_stream(stream), src, dst, n, ld,
                     hg::block_order(nt, n, ld, grid), A, flags);
  return hg::launched("affine_kernel");
}
