// RANSAC hypothesise-and-verify on the GPU.
//
// Two forms of scoring, both of which decide a point in float only where a bound
// on the rounding error proves the decision and leave the rest to a float64
// recount, so that every count is the float64 test's (error_bound in
// ransac_dev.hpp, tile_bound in tile_dev.hpp, which also says what it rests on):
//  * vector form (single pair): each lane holds P correspondences in registers,
//    every lane reads the hypothesis from LDS, the inlier test runs per
//    (hypothesis, point) and counts come from a wavefront ballot + popcount.
//    Its work is split into blocks of few hypotheses, which fills the chip from
//    one pair;
//  * tile form (many pairs): tiles of 32 hypotheses x 32 points on the matrix
//    cores, counts summed in the lanes.
// The argmax is over a packed (count, ~index) key.
//
// Launches:
//  * fused single pair: grid = hypothesis blocks, each workgroup (512 threads)
//    solving and scoring its hypotheses and writing its best key; a second
//    kernel reduces them and writes the mask;
//  * plain single pair: solve all -> H buffer, score, argmax, mask kernels;
//  * batched persistent: CUs x blocks_per_cu workgroups (256 threads) drain an
//    atomic queue of items (pair, block of hypotheses) ordered by pair size
//    (largest first); each item atomicMax-es its key into the pair's; a finish
//    kernel (one workgroup per pair) then recomputes each winner and writes the
//    outputs and masks;
//  * adaptive termination: items are rounds of 64 hypotheses; each writes its
//    round key into a write-once slot and may advance an advisory prefix that
//    lets later rounds be skipped; the finish kernel applies the stopping rule
//    to the slots in order.
// Workgroups exchange nothing but atomics whose results the finish kernel
// reads after the launch boundary, so no fences are needed.
#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <tuple>
#include <vector>

#include "common.hpp"
#include "ransac_dev.hpp"
#include "tile_dev.hpp"

namespace hg {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;
// Waves per workgroup of the fused single-pair kernel: 8 (512 threads, two
// workgroups and four waves per SIMD at about two workgroups per CU).
constexpr int kFusedWaves = 8;

struct RansacArgs {
  const float *corr;
  int64_t ld;
  const int64_t *off;      // n_pairs + 1 offsets, or nullptr for one pair of n_single points
  int32_t n_single;
  int32_t n_pairs;
  int32_t n_hyp;
  int32_t n_hb;            // hypothesis blocks per pair
  int64_t n_items;         // n_pairs * n_hb
  float tau;
  float inv_tau;           // 1/tau rounded to float (the scoring form's scale)
  uint32_t k0, k1;         // Philox key (seed low / high word)
  float *best_H;
  int32_t *best_count;
  int32_t *best_hyp;
  uint8_t *mask;
  int32_t *hyp_counts;     // may be null
  unsigned long long *keys;
  uint32_t *queue;
  const int32_t *order;    // pair processing order (largest first), or nullptr
  float *hbuf;             // single pair: every hypothesis's H (9 floats), or nullptr
  unsigned long long *blockbest;   // single pair: best key of each work item, or nullptr
  // adaptive termination (nullptr pst = off): work items are rounds of HB
  // hypotheses; per pair and round the round's best key (write-once slot);
  // per pair the advisory prefix and stopping hint
  struct PairState *pst;
  unsigned long long *rkey;
  int32_t *iorder;         // adaptive: queue position -> pair * n_hb + round, or NULL
  struct Extent *extent;   // many pairs: centre and reach of each pair's points
  int32_t *n_eval;
  double one_minus_conf;
};

// Advisory state of one pair under adaptive termination, read and written
// only with relaxed atomics. `prefix` = (front << 32) | best count over rounds
// [0, front), extended in order from published round keys (monotone in both
// halves, so atomicMax keeps the furthest one); `stop` = a number of rounds
// after which no round is needed (an exact stopping point or a bound on it;
// atomicMin). Rounds at or past `stop` are skipped or abandoned. Nothing here
// decides a result: the finish kernel re-applies the rule to the published
// round keys in order.
struct PairState {
  unsigned long long prefix;
  uint32_t stop, pad;
};

// Round key slot not yet published (no real key has all bits set).
constexpr unsigned long long kUnpublished = ~0ull;

// Hypotheses per round under adaptive termination (one work item).
constexpr int kRoundHyps = 64;

__device__ __forceinline__ void pair_range(const RansacArgs &a, int p, int64_t &base, uint32_t &n) {
  if (a.off) {
    // clamped into the planes, so that offsets outside them cannot move an access out
    base = min(max(a.off[p], int64_t(0)), a.ld);
    const int64_t e = min(max(a.off[p + 1], base), a.ld);
    const int64_t m = e - base;
    n = m > 0x7FFFFFFF ? 0x7FFFFFFFu : static_cast<uint32_t>(m);
  } else {
    base = 0;
    n = static_cast<uint32_t>(a.n_single);
  }
}

// Maximum of a 64-bit value over the 64 lanes of a wave (result in every lane).
__device__ __forceinline__ unsigned long long wave_max_u64(unsigned long long v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const unsigned long long w = __shfl_xor(v, o);
    v = w > v ? w : v;
  }
  return v;
}

// Maximum of a float over the 64 lanes of a wave (result in every lane).
__device__ __forceinline__ float wave_max_f32(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
  return v;
}

// Rows of points per group in the scoring loop: the unit whose float32
// count is replaced by a float64 recount when a sign in it is not proven.
constexpr int kGroup = 4;

// Groups to recount, listed in LDS by the scoring loop (which leaves their
// points out of its counts) and counted after it, when the loop's point
// registers are free. Entry: the chunk's first point and (hypothesis |
// group << 6 | wave << 9 | rows << 12). n counts every append; past kFixCap
// the list has overflowed and every hypothesis is recounted in float64.
constexpr uint32_t kFixCap = 512;
static_assert(kWaves <= 8 && kFusedWaves <= 8, "a recount entry holds the wave index in 3 bits");
struct FixList {
  uint32_t n;
  uint32_t e[kFixCap][2];
};

// Inliers of H (the float H, given as doubles) among `rows` (<= kGroup) rows
// of 64 points, NW * 64 points apart from point ib of this lane (points
// at or past n excluded), by the float64 test on the operands read from
// memory (every row's loads issued before the first test; 32-bit byte
// offsets from the plane bases, which the pair range keeps below 2^33).
template <int NW>
__device__ __forceinline__ uint32_t count_f64(const RansacArgs &a, const float *X1,
                                              const float *Y1, const float *X2, const float *Y2,
                                              uint32_t ib, uint32_t n, uint32_t rows,
                                              const double *g) {
  float x1[kGroup], y1[kGroup], x2[kGroup], y2[kGroup];
#pragma unroll
  for (int q = 0; q < kGroup; ++q) {
    const uint32_t j = min(ib + q * NW * 64u, n - 1u);   // loads stay inside the pair
    x1[q] = X1[j];
    y1[q] = Y1[j];
    x2[q] = X2[j];
    y2[q] = Y2[j];
  }
  uint32_t c = 0u;
#pragma unroll
  for (int q = 0; q < kGroup; ++q) {
    const uint32_t i = ib + q * NW * 64u;
    const bool in = inlier_f64(g, x1[q], y1[q], x2[q], y2[q], a.tau);
    c += __popcll(__ballot(in && i < n && static_cast<uint32_t>(q) < rows));
  }
  return c;
}

// List length up to which fix_counts recounts every listed group without
// bounding which hypotheses can still reach the best.
constexpr uint32_t kBoundMin = 32;

// After the scoring loop (and a workgroup barrier): apply the listed float64
// recounts to cnt, or on overflow recount every valid hypothesis over all
// points. With `all` false (per-hypothesis counts are not an output), a
// hypothesis is recounted only if it could still reach the best count among
// the hypotheses counted exactly here: its listed points added to its count
// reach that best (ties included). The others keep a count below their true
// one, which stays below the best, so the maximum, its lowest index and the
// mask do not change. The bound costs two barriers and LDS atomics, so with
// at most kBoundMin entries every listed group is recounted instead. ub: LDS
// scratch of HB words. NW: waves per workgroup. Ends with a workgroup barrier.
template <int NW>
__device__ void fix_counts(const RansacArgs &a, int64_t base, uint32_t n, const double (*H0s)[9],
                           FixList *fx, uint64_t vmask, int nh, uint32_t *cnt, bool all,
                           uint32_t *ub) {
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const float *X1 = a.corr + base, *Y1 = a.corr + a.ld + base;
  const float *X2 = a.corr + 2 * a.ld + base, *Y2 = a.corr + 3 * a.ld + base;
  const uint32_t ne = fx->n;
  if (ne <= kFixCap) {
    uint32_t best = 0u;
    const bool bound = !all && ne > kBoundMin;
    if (bound) {
      // ub[h]: the count so far plus the listed points of h
      for (int h = threadIdx.x; h < nh; h += NW * 64) ub[h] = cnt[h];
      __syncthreads();
      for (uint32_t k = threadIdx.x; k < ne; k += NW * 64) {
        const uint32_t w = fx->e[k][1];
        atomicAdd(&ub[w & 63u], ((w >> 12) & 31u) * 64u);
      }
      __syncthreads();
      // the best exact count: valid hypotheses with nothing listed
      const bool exact = lane < nh && ((vmask >> lane) & 1ull) && ub[lane] == cnt[lane];
      uint32_t v = exact ? cnt[lane] : 0u;
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) v = max(v, static_cast<uint32_t>(__shfl_xor(v, o)));
      best = v;
    }
    for (uint32_t k = wave; k < ne; k += NW) {
      const uint32_t c0 = fx->e[k][0], w = fx->e[k][1];
      const uint32_t h = w & 63u, g = (w >> 6) & 7u, wv = (w >> 9) & 7u, rows = (w >> 12) & 31u;
      if (bound && ub[h] < best) continue;   // cannot reach the best
      const uint32_t ib = c0 + (g * kGroup * NW + wv) * 64u + lane;
      const uint32_t c64 = count_f64<NW>(a, X1, Y1, X2, Y2, ib, n, rows, H0s[h]);
      if (lane == 0 && c64) atomicAdd(&cnt[h], c64);
    }
  } else {
    for (int h = wave; h < nh; h += NW) {
      if (!((vmask >> h) & 1ull)) continue;
      uint32_t c = 0u;
      for (uint32_t c0 = 0; c0 < n; c0 += NW * 64u * kGroup)
        for (int wv = 0; wv < NW; ++wv)
          c += count_f64<NW>(a, X1, Y1, X2, Y2, c0 + wv * 64u + lane, n, kGroup, H0s[h]);
      if (lane == 0) cnt[h] = c;
    }
  }
  __syncthreads();
}

// Count, for each hypothesis h < nh whose bit is set in vmask, the inliers
// among the points [base, base + n) held in registers (P per lane); each wave
// adds its counts into cnt[h] (LDS atomics). Hs holds the hypotheses' scoring
// forms. TAIL: the chunk runs past n and lanes beyond it are masked out of the
// ballots.
// Each wave decides its P x 64 points in float32, in groups of kGroup rows,
// and keeps per lane and group the minimum over its points of
// |e32| - |w| k1; where that reaches k0 for some lane (a point whose float32
// sign is not proven, see error_bound), the group is listed in fx for a
// float64 recount after the loop (fix_counts). The error bound's magnitudes
// are the wave's maxima over its points, and its coefficients are computed
// once per chunk, lane h for hypothesis h.
template <int P, bool TAIL, int NW>
__device__ __forceinline__ void score_chunk(const RansacArgs &a, const float *X1, const float *Y1,
                                            const float *X2, const float *Y2, uint32_t c0,
                                            uint32_t n, const float (*Hs)[9],
                                            uint64_t vmask, int nh, uint32_t *cnt,
                                            FixList *fx) {
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  float x1[P], y1[P], x2[P], y2[P];
  uint64_t live[TAIL ? P : 1];
  float m1 = 0.0f, m2 = 0.0f, m3 = 0.0f, m4 = 0.0f;
#pragma unroll
  for (int p = 0; p < P; ++p) {
    const uint32_t i = c0 + (p * NW + wave) * 64 + lane;
    const uint32_t j = (TAIL && i >= n) ? n - 1u : i;   // every load stays inside the pair
    x1[p] = X1[j];
    y1[p] = Y1[j];
    x2[p] = X2[j] * a.inv_tau;
    y2[p] = Y2[j] * a.inv_tau;
    if (TAIL) live[p] = __ballot(i < n);
    m1 = fmaxf(m1, fabsf(x1[p]));
    m2 = fmaxf(m2, fabsf(y1[p]));
    m3 = fmaxf(m3, fabsf(x2[p]));
    m4 = fmaxf(m4, fabsf(y2[p]));
  }
  m1 = wave_max_f32(m1);
  m2 = wave_max_f32(m2);
  m3 = wave_max_f32(m3);
  m4 = wave_max_f32(m4);
  // lane h: error-bound coefficients of hypothesis h over this wave's points
  float k1v = 0.0f, k0v = 0.0f;
  if (lane < nh) error_bound(Hs[lane], m1, m2, m3, m4, k1v, k0v);
  for (int h = 0; h < nh; ++h) {
    if (!((vmask >> h) & 1ull)) continue;
    // H read from LDS by every lane (one address: a broadcast) and used from
    // vector registers; scalar copies would cost a readfirstlane per entry and
    // moves wherever an FMA needs two of them
    float hh[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) hh[k] = Hs[h][k];
    const float k1 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(k1v), h));
    const float k0 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(k0v), h));
    // rows in groups of kGroup: per group the float32 count and the minimum
    // over its points of |e32| - |w| k1 (the margin by which the sign is
    // proven); a group with a sign not proven is listed for a float64 recount
    // (which then supplies its whole count) instead of counted here
    uint32_t c = 0;
#pragma unroll
    for (int g = 0; g < (P + kGroup - 1) / kGroup; ++g) {
      uint32_t cg = 0u;
      float slack = __builtin_inff();
#pragma unroll
      for (int q = 0; q < kGroup; ++q) {
        const int p = g * kGroup + q;
        if (p < P) {
          float w;
          const float e = test_f32(hh, x1[p], y1[p], x2[p], y2[p], w);
          uint64_t m = __ballot(e <= 0.0f);
          if (TAIL) m &= live[p];
          cg += __popcll(m);
          slack = fminf(slack, fmaf(-fabsf(w), k1, fabsf(e)));
        }
      }
      if (__builtin_expect(__ballot(slack <= k0) != 0ull, 0)) {
        if (lane == 0) {
          const uint32_t k = atomicAdd(&fx->n, 1u);
          if (k < kFixCap) {
            const uint32_t rows = min(kGroup, P - g * kGroup);
            fx->e[k][0] = c0;
            fx->e[k][1] = static_cast<uint32_t>(h) | (static_cast<uint32_t>(g) << 6) |
                          (static_cast<uint32_t>(wave) << 9) | (rows << 12);
          }
        }
      } else {
        c += cg;
      }
    }
    if (lane == 0 && c) atomicAdd(&cnt[h], c);
  }
}

// Full chunks of P points per lane, then one masked tail chunk of just enough 64-point rows per wave (1 to 8), so that a
// pair's last chunk leaves fewer than NW x 64 lane slots idle (NW: waves per
// workgroup). Counts are integer sums over the points, so the result does not
// depend on the chunking.
template <int P, int NW = kWaves>
__device__ __forceinline__ void score_hyps(const RansacArgs &a, int64_t base, uint32_t n,
                                           const float (*Hs)[9], uint64_t vmask, int nh,
                                           uint32_t *cnt, FixList *fx) {
  static_assert(P == 8, "the tail has at most 8 rows");
  const float *X1 = a.corr + base, *Y1 = a.corr + a.ld + base;
  const float *X2 = a.corr + 2 * a.ld + base, *Y2 = a.corr + 3 * a.ld + base;
  constexpr uint32_t kChunk = NW * 64 * P;
  uint32_t c0 = 0;
  for (; c0 + kChunk <= n; c0 += kChunk)
    score_chunk<P, false, NW>(a, X1, Y1, X2, Y2, c0, n, Hs, vmask, nh, cnt, fx);
  if (c0 < n) {
    // fewer than kChunk points remain: 1 .. 8 rows of 64 points per wave
    const uint32_t rows = (n - c0 + 63u) / 64u;
    switch ((rows + NW - 1) / NW) {
#define HG_TAIL(R) \
  case R:          \
    score_chunk<R, true, NW>(a, X1, Y1, X2, Y2, c0, n, Hs, vmask, nh, cnt, fx); \
    break;
      HG_TAIL(1)
      HG_TAIL(2)
      HG_TAIL(3)
      HG_TAIL(4)
      HG_TAIL(5)
      HG_TAIL(6)
      HG_TAIL(7)
      default:
        score_chunk<8, true, NW>(a, X1, Y1, X2, Y2, c0, n, Hs, vmask, nh, cnt, fx);
#undef HG_TAIL
    }
  }
}

// ---- scoring on the matrix cores (many pairs) --------------------------------
// A wave scores tiles of 32 hypotheses x 32 points. u, v and w of a tile (the
// rows of the scoring form times (x1, y1, 1)) come from one
// v_mfma_f32_32x32x16_bf16 each: a float is exactly the sum of three bfloat16
// pieces, and the six products of pieces that reach 2^-22 of a term, for x1 and
// y1, and the three pieces of the constant fill 15 of the 16 slots of K:
//   point       x0 x0 x1 x1 x0 x2 | 1 1    y0 y0 y1 y1 y0 y2 | 1 0
//   hypothesis  g0 g1 g0 g1 g2 g0 | c0 c1  (the same for y)  | c2 0
// Lane l holds slots 8 (l / 32) .. + 7 of hypothesis (operand A) or point
// (operand B) l % 32, and gets hypothesis m = 8 (i / 4) + 4 (l / 32) + i % 4 of
// point l % 32 in result i.
// The rest runs in float on the results, 7 instructions per element:
//   ru = u - x2c w, rv = v - y2c w, t = clamp(w^2 - (rv^2 + (ru^2 - 0.5)))
// with the rows scaled by sigma so that the error bound of e = ru^2 + rv^2 - w^2
// becomes 0.5: t = 1 proves an inlier, t = 0 an outlier, and anything between
// leaves the point open. Sums of t and t^2 per lane count the inliers and show
// by their difference whether a point was open (0 and 1 are their own squares),
// so counting needs neither compares nor ballots. Every TB tiles a lane
// whose sums differ lists its points (one column of the block) for a float64
// recount and leaves them out. Sums can also agree by rounding with a t just off
// 0 or 1 among them: the difference, the sum of t (1 - t), is then within their
// roundings, 2 TB halves of a last place of at most TB, so such t are within 2^-13
// of 0 or 1, which the slack of the bound covers, and the sum of t within 2^-12 of
// the whole number that it stands for, to which adding it to the total rounds it
// (block_total).
//
// What bounds it: vector issue and the clock that the power limit leaves (1.95
// GHz measured). Of gfx950's vector instructions only float add, mul, FMA (no
// scalar operand, not all three sources in one register bank), 32-bit integer
// add and logic issue every 2 cycles per wave, and compares, min / max and
// conversions every 4; matrix instructions do not overlap them. Per 64
// (hypothesis, point) pairs the vector form (score_chunk) spends 12 float
// instructions, a compare, the minimum and the per-hypothesis overheads, 52
// cycles of 2.4 GHz in all; here 7 float instructions and 1/16 of the three
// MFMAs (33 cycles each), 31 - 35 cycles. For v and w, A holds hypothesis
// (l % 32) ^ 1, so that results i of u and i ^ 1 of v and w belong together:
// the three results start at even registers, and equal indices would put all
// sources of the squares into one bank (35.5 against 31.4 cycles).
// A hypothesis for the tile form: its float H, solver flags, and the rows g that
// go into operand A (centred, scaled by 1/tau and sigma). full: without a bound, to be
// counted in float64 throughout. An invalid, missing or full one gets u = 1024,
// v = w = 0: no inlier and nothing open anywhere.
__device__ __forceinline__ uint32_t tile_hypothesis(const RansacArgs &a, int64_t base, uint32_t n,
                                                    int p, int hyp, bool live, float *h,
                                                    double *g, bool &full) {
  uint32_t f = kZeroH;
  if (live)
    f = make_hypothesis(a.corr, a.ld, base, n, a.k0, a.k1, static_cast<uint32_t>(hyp),
                        static_cast<uint32_t>(p), h);
  full = false;
  if (f == 0u) {
    // rows on coordinates about the pair's centre: halves the magnitudes, and
    // with them the error bound and the points that stay open
    const Extent x = a.extent[p];
    const double it = static_cast<double>(a.inv_tau);
#pragma unroll
    for (int r = 2; r >= 0; --r) {
      const double scale = r == 2 ? 1.0 : it, k = r == 2 ? 0.0 : static_cast<double>(x.k2[r]);
      const double h0 = h[3 * r], h1 = h[3 * r + 1];
      const double h2 = h[3 * r + 2] + (h0 * x.c1[0] + h1 * x.c1[1]);
      g[3 * r] = r == 2 ? h0 : h0 * scale - k * g[6];
      g[3 * r + 1] = r == 2 ? h1 : h1 * scale - k * g[7];
      g[3 * r + 2] = r == 2 ? h2 : h2 * scale - k * g[8];
    }
    float bound;
    full = !tile_bound(g, x, bound);
    // bound sigma^2 = 0.5 (to a rounding or two of the reciprocal root)
    const double sigma = static_cast<double>(__builtin_amdgcn_rsqf(2.0f * bound));
    double top = 0.0;
#pragma unroll
    for (int k = 0; k < 9; ++k) {
      g[k] *= sigma;
      top = fmax(top, fabs(g[k]));
    }
    full |= !(top < kMaxEntry);
  }
  if (f != 0u || full)
#pragma unroll
    for (int k = 0; k < 9; ++k) g[k] = k == 2 ? 1024.0 : 0.0;
  return f;
}

// Points whose decision is open, listed by the tile loop: the first of their
// tiles and hypothesis | column << 6 | number of tiles << 11. n counts every
// append; the hypotheses (bit m of lost) of those past the capacity are counted
// in float64 throughout.
template <int CAP>
struct OpenList {
  uint32_t n;
  uint32_t lost[2];
  uint32_t e[CAP][2];
};

// The lane number, opaque to the compiler: what is computed from it stays where
// it is used. Hoisted out of the persistent loop, such values (LDS addresses,
// mostly) exceed the registers beside the tile loop's and cost scratch reloads
// in every item.
__device__ __forceinline__ uint32_t lane_here() {
  uint32_t lane = threadIdx.x & 63u;
  asm volatile("" : "+v"(lane));
  return lane;
}

// Score the 32 hypotheses of operands au, av, aw (numbers m0 .. m0 + 31 in the
// item) against tiles [t0, t1) of a segment of n points, whose first tile is
// number first_tile of the pair; adds the inliers to tot (by result and lane;
// block_total) and lists open points. Returns false if the item is abandoned (adaptive:
// round hb is at or past the stopping hint, checked once per block of tiles).
template <int TB, int CAP>
__device__ __forceinline__ bool score_tiles(const RansacArgs &a, const float *X1, const float *Y1,
                                            const float *X2, const float *Y2, uint32_t n,
                                            uint32_t t0, uint32_t t1, uint32_t first_tile,
                                            uint32_t m0, bf16x8 au, bf16x8 av, bf16x8 aw,
                                            const Extent &x, float (*tot)[64],
                                            OpenList<CAP> &open,
                                            const uint32_t *stop, uint32_t hb) {
  const int lane = lane_here(), col = lane & 31, half = lane >> 5;
  const float *C = half ? Y1 : X1;
  const uint32_t one = half ? 0x00003f80u : 0x3f803f80u;
  // in registers of their own: a scalar operand would halve the rate
  float it = a.inv_tau, cc = half ? x.c1[1] : x.c1[0], kx = x.k2[0], ky = x.k2[1];
  asm volatile("" : "+v"(it), "+v"(cc), "+v"(kx), "+v"(ky));
  const uint32_t part_tile = n / 32u;   // the segment's partial tile, if it has one
  const float part_ky = static_cast<uint32_t>(col) < n % 32u ? ky : __builtin_nanf("");
  // coordinates of this lane's point of tile t, the index clamped into the segment
  auto load = [&](uint32_t t, float &c, float &x2, float &y2) {
    if (t < part_tile) {
      const uint32_t at = t * 32u;   // scalar: only col is per lane
      c = (C + at)[col];
      x2 = (X2 + at)[col];
      y2 = (Y2 + at)[col];
    } else {
      const uint32_t at = min(t * 32u + col, n - 1u);
      c = C[at];
      x2 = X2[at];
      y2 = Y2[at];
    }
  };
  float c, x2, y2;
  load(t0, c, x2, y2);
  for (uint32_t b0 = t0; b0 < t1; b0 += TB) {
    if (stop &&
        hb >= __hip_atomic_load(stop, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
      return false;
    const uint32_t b1 = min(b0 + TB, t1);
    f32x16 s = {}, q = {};
    for (uint32_t t = b0; t < b1; ++t) {
      // past the last point of the segment: a NaN in y2c, so that t = 0
      const float kt = t == part_tile ? part_ky : ky;
      float cn, x2n, y2n;
      load(t + 1u, cn, x2n, y2n);
      const bf16x8 b = point_operand(c - cc, one);
      const f32x16 zero = {};
      const f32x16 u = __builtin_amdgcn_mfma_f32_32x32x16_bf16(au, b, zero, 0, 0, 0);
      const f32x16 w = __builtin_amdgcn_mfma_f32_32x32x16_bf16(aw, b, zero, 0, 0, 0);
      const f32x16 v = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, b, zero, 0, 0, 0);
      const float xc = fmaf(x2, it, -kx), yc = fmaf(y2, it, -kt);
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const float wj = w[i ^ 1];
        const float ru = fmaf(-xc, wj, u[i]);
        const float rv = fmaf(-yc, wj, v[i ^ 1]);
        const float d = fmaf(rv, rv, fmaf(ru, ru, -0.5f));
        // clamp to [0, 1], NaN to 0 (an output modifier of the FMA)
        const float in = __builtin_amdgcn_fmed3f(fmaf(wj, wj, -d), 0.0f, 1.0f);
        s[i] += in;
        q[i ^ 1] = fmaf(in, in, q[i ^ 1]);
      }
      // whole register groups, so that q[i ^ 1] is not in the bank of result i
      asm volatile("" : "+v"(s), "+v"(q));
      c = cn;
      x2 = x2n;
      y2 = y2n;
    }
    uint64_t any = 0ull;
#pragma unroll
    for (int i = 0; i < 16; ++i) any |= __ballot(s[i] != q[i ^ 1]);
    if (any != 0ull) {
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        if (s[i] != q[i ^ 1]) {
          const uint32_t m = m0 + 8u * (i / 4) + 4u * half + i % 4;
          const uint32_t k = atomicAdd(&open.n, 1u);
          if (k < CAP) {
            open.e[k][0] = first_tile + b0;
            open.e[k][1] = m | (static_cast<uint32_t>(col) << 6) | ((b1 - b0) << 11);
          } else {
            atomicOr(&open.lost[m >> 5], 1u << (m & 31u));
          }
          s[i] = 0.0f;
        }
      }
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) tot[i][lane] = block_total(tot[i][lane], s[i]);
  }
  return true;
}

// Adaptive stopping rule: with eps = best_count / n, enough samples have been
// drawn once (1 - eps^4)^m <= 1 - confidence, i.e. m >= log(1 - confidence) /
// log(1 - eps^4) rounded up (m integer). The power is taken by repeated
// squaring in double.
__device__ __forceinline__ bool enough_samples(uint32_t best_count, uint32_t n, uint32_t m,
                                               double one_minus_conf) {
  if (n == 0u) return false;
  const double eps = static_cast<double>(best_count) / static_cast<double>(n);
  const double e2 = eps * eps;
  const double q = 1.0 - e2 * e2;
  double r = 1.0, b = q;
  for (uint32_t e = m; e; e >>= 1) {
    if (e & 1u) r *= b;
    b *= b;
  }
  return r <= one_minus_conf;
}

#define HG_AGENT __HIP_MEMORY_SCOPE_AGENT

__device__ __forceinline__ uint32_t key_count(unsigned long long k) {
  return k ? static_cast<uint32_t>((k >> 32) - 1ull) : 0u;
}

// Called by one thread after round hb of pair p published `key`. If hb is the
// pair's front, extends the merged prefix over the rounds published since
// (in order), applies the stopping rule at each step, and lowers `stop` to
// the stopping point when it holds, else to the bound that the prefix's best
// count gives (the count only grows and the rule is monotone in it, so the
// rule holds at the latest there). Every value read is final (a slot is
// written once per launch) or the sentinel, so a stale read only means a
// shorter prefix, never a wrong one.
__device__ void adaptive_hint(const RansacArgs &a, int p, uint32_t n_pts, int HB, int hb,
                              unsigned long long key) {
  PairState *st = a.pst + p;
  const unsigned long long w = __hip_atomic_load(&st->prefix, __ATOMIC_RELAXED, HG_AGENT);
  uint32_t f = static_cast<uint32_t>(w >> 32);
  if (f != static_cast<uint32_t>(hb)) return;
  uint32_t bc = static_cast<uint32_t>(w);
  uint32_t s = __hip_atomic_load(&st->stop, __ATOMIC_RELAXED, HG_AGENT);
  const uint32_t n_hyp = static_cast<uint32_t>(a.n_hyp);
  const unsigned long long *rk = a.rkey + static_cast<int64_t>(p) * a.n_hb;
  unsigned long long k = key;
  for (;;) {
    bc = max(bc, key_count(k));
    ++f;
    const uint32_t m = min(f * static_cast<uint32_t>(HB), n_hyp);
    if (m >= n_hyp || enough_samples(bc, n_pts, m, a.one_minus_conf)) {
      s = min(s, f);
      break;
    }
    if (f >= s) break;
    k = __hip_atomic_load(&rk[f], __ATOMIC_RELAXED, HG_AGENT);
    if (k == kUnpublished) break;
  }
  for (uint32_t c = f + 1u; c < s; ++c)
    if (enough_samples(bc, n_pts, min(c * static_cast<uint32_t>(HB), n_hyp), a.one_minus_conf)) {
      s = c;
      break;
    }
  atomicMax(&st->prefix, (static_cast<unsigned long long>(f) << 32) | bc);
  atomicMin(&st->stop, s);
}

// Pair and round or hypothesis block of a work item: pair-major (all blocks of
// the largest pair first), or under adaptive termination in the staggered
// round order (ransac_round_order_kernel) or round-major.
__device__ __forceinline__ void item_place(const RansacArgs &a, int64_t item, int &p, int &hb) {
  const bool adaptive = a.pst != nullptr;
  if (adaptive && a.iorder) {
    // decoded into range
    const uint32_t code = static_cast<uint32_t>(a.iorder[item]);
    p = min(static_cast<int>(code / static_cast<uint32_t>(a.n_hb)), a.n_pairs - 1);
    hb = static_cast<int>(code % static_cast<uint32_t>(a.n_hb));
  } else {
    const int r = static_cast<int>(adaptive ? item % a.n_pairs : item / a.n_hb);
    hb = static_cast<int>(adaptive ? item / a.n_pairs : item % a.n_hb);
    p = a.order ? a.order[r] : r;
  }
}

// Inliers of hypothesis lane % 32 over the tile loop's totals, in every lane:
// lane l adds 16 of the 32 columns (rotated, so that the lanes of a bank read
// different words).
__device__ __forceinline__ uint32_t tile_count(const float (*tot)[64]) {
  const int lane = lane_here();
  const int m = lane & 31, i = (m >> 3) * 4 + (m & 3), h = (m >> 2) & 1;
  uint32_t c = 0u;
#pragma unroll
  for (int k = 0; k < 16; ++k)
    c += total_count(tot[i][32 * h + 16 * (lane >> 5) + ((k + m) & 15)]);
  return c + __shfl_xor(c, 32);
}

// The float64 test with H in memory as floats.
__device__ __forceinline__ bool inlier_of(const float *H, float x1, float y1, float x2, float y2,
                                          float tau) {
  double g[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) g[k] = H[k];
  return inlier_f64(g, x1, y1, x2, y2, tau);
}

// Float64 recount of a list's entries first, first + step, ... by one wave, TB
// lanes to an entry; added to cnt.
template <int TB, int CAP>
__device__ __forceinline__ void count_open(const RansacArgs &a, const float *X1, const float *Y1,
                                           const float *X2, const float *Y2, uint32_t n,
                                           const float (*H)[9], const OpenList<CAP> &open,
                                           uint32_t first, uint32_t step, uint32_t *cnt) {
  const uint32_t lane = lane_here();
  constexpr uint32_t kPer = 64u / TB;   // entries at a time
  const uint32_t ne = min(open.n, static_cast<uint32_t>(CAP));
  for (uint32_t k0 = first * kPer; k0 < ne; k0 += step * kPer) {
    const uint32_t k = k0 + lane / TB;
    bool in = false;
    uint32_t h = 0u;
    if (k < ne) {
      const uint32_t w = open.e[k][1];
      h = w & 63u;
      const uint32_t j = lane % TB;
      const uint32_t i = (open.e[k][0] + j) * 32u + ((w >> 6) & 31u);
      if (j < ((w >> 11) & 63u) && i < n) in = inlier_of(H[h], X1[i], Y1[i], X2[i], Y2[i], a.tau);
    }
    const uint64_t b = __ballot(in) >> (lane / TB * TB);
    if (lane % TB == 0u && k < ne) {
      const uint32_t c = __popcll(b & ((1ull << TB) - 1ull));
      if (c) atomicAdd(&cnt[h], c);
    }
  }
}

// Float64 inliers of H among all points of the pair, by one wave.
__device__ __forceinline__ uint32_t count_all(const RansacArgs &a, const float *X1, const float *Y1,
                                              const float *X2, const float *Y2, uint32_t n,
                                              const float *H) {
  const uint32_t lane = lane_here();
  uint32_t c = 0u;
  for (uint32_t i = 0u; i < n; i += 64u) {
    const uint32_t j = i + lane;
    const uint32_t k = min(j, n - 1u);
    c += __popcll(__ballot(inlier_of(H, X1[k], Y1[k], X2[k], Y2[k], a.tau) && j < n));
  }
  return c;
}

// Points per segment of the tile loop: 32-bit point offsets, and per-lane totals
// below 2^23.
constexpr uint32_t kSegment = 1u << 28;

// One item of the queue, placed: filled by one lane, read by the workgroup.
struct ItemSlot {
  int64_t item, base;
  int32_t p, hb;
  uint32_t n, skip;
};

// Shared memory of a workgroup of the many-pair kernel, whose kWaves waves take an
// item together.
constexpr int kGroupOpen = 1024;
template <int HB>
struct TileSmem {
  static constexpr int HT = (HB + 31) / 32;
  u32x4 op[HT][3][64];     // operand A of the three rows, by lane
  float H0[HB][9];         // the float H (for the float64 test)
  uint32_t valid[HB];
  uint32_t full[HB];       // 1: counted in float64 throughout
  uint32_t cnt[HB];
  float tot[kWaves][16][64];   // per wave: inliers by result and lane, above kTotalZero
  OpenList<kGroupOpen> open;
  ItemSlot slot[2];
};

// Takes the next item from the queue (one lane).
__device__ __forceinline__ void fetch_item(const RansacArgs &a, ItemSlot &s) {
  const int64_t item = static_cast<int64_t>(atomicAdd(a.queue, 1u));
  int p = 0, hb = 0;
  int64_t base = 0;
  uint32_t n = 0u;
  if (item < a.n_items) {
    item_place(a, item, p, hb);
    pair_range(a, p, base, n);
  }
  s.item = item;
  s.base = base;
  s.p = p;
  s.hb = hb;
  s.n = n;
}

// Step 1, one wave: solve the item's hypotheses, one per lane, and lay out their
// operands. Under adaptive termination a round at or past a known stopping
// point is not evaluated (skip).
template <int HB>
__device__ __forceinline__ void group_solve(const RansacArgs &a, int64_t base, uint32_t n, int p,
                                            int hb, TileSmem<HB> &sm, uint32_t &skip) {
  const int t = lane_here();
  const bool past = a.pst && static_cast<uint32_t>(hb) >=
                                 __hip_atomic_load(&a.pst[p].stop, __ATOMIC_RELAXED, HG_AGENT);
  if (t == 0) skip = past ? 1u : 0u;
  if (past || t >= 32 * TileSmem<HB>::HT) return;
  float h[9];
  double g[9];
  bool full;
  const uint32_t f =
      tile_hypothesis(a, base, n, p, hb * HB + t, t < min(HB, a.n_hyp - hb * HB), h, g, full);
#pragma unroll
  for (int r = 0; r < 3; ++r) {
    float x[3][3];
#pragma unroll
    for (int k = 0; k < 3; ++k) pieces(static_cast<float>(g[3 * r + k]), x[k]);
    const int c = (t & 31) ^ (r ? 1 : 0);
    sm.op[t >> 5][r][c] = row_operand(x[0], x[2], 0);
    sm.op[t >> 5][r][c + 32] = row_operand(x[1], x[2], 1);
  }
  if (t < HB) {
    if (f == 0u)
#pragma unroll
      for (int k = 0; k < 9; ++k) sm.H0[t][k] = h[k];
    sm.valid[t] = f == 0u ? 1u : 0u;
    sm.full[t] = full ? 1u : 0u;
    sm.cnt[t] = 0u;
  }
  if (t == 0) sm.open.n = sm.open.lost[0] = sm.open.lost[1] = 0u;
}

// Step 2, every wave: its share of the pair's tiles against every hypothesis.
template <int TB, int HB>
__device__ __forceinline__ void group_score(const RansacArgs &a, int64_t base, uint32_t n, int p,
                                            int hb, int wave, TileSmem<HB> &sm) {
  const float *X1 = a.corr + base, *Y1 = a.corr + a.ld + base;
  const float *X2 = a.corr + 2 * a.ld + base, *Y2 = a.corr + 3 * a.ld + base;
  const uint32_t *stop = a.pst ? &a.pst[p].stop : nullptr;
  const int lane = lane_here();
  for (uint32_t seg = 0; seg < n; seg += kSegment) {
    const uint32_t ns = min(n - seg, kSegment);
    const uint32_t tiles = (ns + 31u) / 32u, share = (tiles + kWaves - 1u) / kWaves;
    const uint32_t t0 = min(static_cast<uint32_t>(wave) * share, tiles), t1 = min(t0 + share, tiles);
    for (int ht = 0; ht < TileSmem<HB>::HT && t0 < t1; ++ht) {
#pragma unroll
      for (int i = 0; i < 16; ++i) sm.tot[wave][i][lane] = kTotalZero;
      if (!score_tiles<TB>(a, X1 + seg, Y1 + seg, X2 + seg, Y2 + seg, ns, t0, t1, seg / 32u,
                           32u * ht, __builtin_bit_cast(bf16x8, sm.op[ht][0][lane]),
                           __builtin_bit_cast(bf16x8, sm.op[ht][1][lane]),
                           __builtin_bit_cast(bf16x8, sm.op[ht][2][lane]), a.extent[p],
                           sm.tot[wave], sm.open, stop, static_cast<uint32_t>(hb)))
        return;
      const uint32_t c = tile_count(sm.tot[wave]);
      if (lane < 32 && 32 * ht + lane < HB && c) atomicAdd(&sm.cnt[32 * ht + lane], c);
    }
  }
}

// Step 4, wave 0: an item's counts and its best key; c and ok: count and
// validity of hypothesis hb HB + lane. Under adaptive termination a wave may
// have given the round up: then it is at or past the stopping round (which
// only decreases), and nothing of it is published.
template <int HB>
__device__ __forceinline__ void group_publish(const RansacArgs &a, int p, int hb, uint32_t n,
                                              uint32_t c, bool ok) {
  const int t = lane_here();
  if (a.pst && static_cast<uint32_t>(hb) >=
                   __hip_atomic_load(&a.pst[p].stop, __ATOMIC_RELAXED, HG_AGENT))
    return;
  const int h = hb * HB + t;
  if (a.hyp_counts && t < HB && h < a.n_hyp)
    a.hyp_counts[static_cast<int64_t>(p) * a.n_hyp + h] = ok ? static_cast<int32_t>(c) : 0;
  const unsigned long long key = wave_max_u64(ok ? pack_key(c, static_cast<uint32_t>(h)) : 0ull);
  if (t != 0) return;
  if (a.pst) {
    // write-once slot, then the advisory prefix / stopping hint
    __hip_atomic_store(&a.rkey[static_cast<int64_t>(p) * a.n_hb + hb], key, __ATOMIC_RELAXED,
                       HG_AGENT);
    adaptive_hint(a, p, n, HB, hb, key);
  } else if (key != 0ull) {
    atomicMax(&a.keys[p], key);  // the pair's outputs come from the finish kernel
  }
}

// A persistent workgroup of any many-pair launch: its waves take items of HB
// hypotheses of one pair together. In the fixed-count form an item's serial steps run beside each other: while one of waves 1 - 3 solves its
// hypotheses, another takes the next item from the queue and wave 0 publishes
// the item before. Adaptive rounds are published at once, and the next is taken
// only then (taken ahead, 512 pairs of up to 8000 points: 382 us, not 337, by
// rounds that a fresher stopping hint would have skipped). Every lane-divergent
// region is followed by a barrier before the loop closes, and every wave passes
// the same barriers: the conditions around them are slot values read by all
// after a barrier.
template <int TB, int HB>
__device__ __forceinline__ void group_loop(const RansacArgs &a, TileSmem<HB> &sm) {
  const int lane = threadIdx.x & 63;
  // scalar, so that the tile loop's counters and branches are
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
  // different waves for workgroups that share a compute unit (and its SIMDs)
  const int turn = static_cast<int>((blockIdx.x >> 8) % 3u);
  const int solver = 1 + turn, fetcher = 1 + (turn + 1) % 3;
  if (threadIdx.x == 0) fetch_item(a, sm.slot[0]);
  __syncthreads();
  // the item that wave 0 has yet to publish
  int wait_p = -1, wait_hb = 0;
  uint32_t wait_n = 0u, wait_c = 0u;
  bool wait_ok = false;
  for (int cur = 0;; cur ^= 1) {
    const ItemSlot s = sm.slot[cur];
    if (__builtin_amdgcn_readfirstlane(s.item >= a.n_items ? 1 : 0)) break;
    const int p = __builtin_amdgcn_readfirstlane(s.p), hb = __builtin_amdgcn_readfirstlane(s.hb);
    const uint32_t n = __builtin_amdgcn_readfirstlane(s.n);
    const int64_t base = static_cast<int64_t>(
        (static_cast<uint64_t>(static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(
             static_cast<int>(s.base >> 32)))) << 32) |
        static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(s.base))));
    if (wave == solver) {
      group_solve<HB>(a, base, n, p, hb, sm, sm.slot[cur].skip);
    } else if (wave == fetcher) {
      if (lane == 0 && !a.pst) fetch_item(a, sm.slot[cur ^ 1]);
    } else if (wave == 0 && wait_p >= 0) {
      group_publish<HB>(a, wait_p, wait_hb, wait_n, wait_c, wait_ok);
      wait_p = -1;
    }
    __syncthreads();
    if (__builtin_amdgcn_readfirstlane(sm.slot[cur].skip) == 0u) {
      group_score<TB, HB>(a, base, n, p, hb, wave, sm);
      __syncthreads();
      // 3. float64 counts: the listed points, then the hypotheses without a bound
      // or with points lost to the list (after a barrier: they replace the counts)
      const float *X1 = a.corr + base, *Y1 = a.corr + a.ld + base;
      const float *X2 = a.corr + 2 * a.ld + base, *Y2 = a.corr + 3 * a.ld + base;
      count_open<TB>(a, X1, Y1, X2, Y2, n, sm.H0, sm.open, static_cast<uint32_t>(wave), kWaves,
                     sm.cnt);
      __syncthreads();
      const int nh = min(HB, a.n_hyp - hb * HB), t = lane < HB ? lane : 0;
      for (uint64_t hm = __ballot(lane < nh && (sm.full[t] != 0u ||
                                                ((sm.open.lost[t >> 5] >> (t & 31)) & 1u) != 0u));
           hm; hm &= hm - 1ull) {
        const int h = __ffsll(static_cast<long long>(hm)) - 1;
        if (h % kWaves != wave) continue;
        const uint32_t c = count_all(a, X1, Y1, X2, Y2, n, sm.H0[h]);
        if (lane == 0) sm.cnt[h] = c;
      }
      __syncthreads();
      if (wave == 0) {
        const uint32_t c = sm.cnt[t];
        const bool ok = lane < nh && sm.valid[t] != 0u;
        if (a.pst) {
          group_publish<HB>(a, p, hb, n, c, ok);
        } else {
          wait_p = p;
          wait_hb = hb;
          wait_n = n;
          wait_c = c;
          wait_ok = ok;
        }
      }
    }
    if (a.pst && threadIdx.x == 0) fetch_item(a, sm.slot[cur ^ 1]);
    __syncthreads();
  }
  if (wave == 0 && wait_p >= 0) group_publish<HB>(a, wait_p, wait_hb, wait_n, wait_c, wait_ok);
}

// Shared memory of one workgroup of the fused single pair.
template <int HB>
struct Smem {
  float H[HB][9];          // scoring form (rows 1-2 scaled by 1/tau)
  double H0[HB][9];        // the float H, as doubles (for the float64 test)
  uint32_t valid[HB];
  uint32_t cnt[HB];
  uint32_t ub[HB];         // scratch of fix_counts
  FixList fix;             // groups to recount in float64
};

// Process one work item of the fused single pair: hypothesis block hb of HB
// hypotheses (NW waves).
template <int P, int HB, int NW>
__device__ void run_item(const RansacArgs &a, int hb, Smem<HB> &sm) {
  const uint32_t n = static_cast<uint32_t>(a.n_single);
  const int h0 = hb * HB;
  const int nh = min(HB, a.n_hyp - h0);
  // 1. solve this block's hypotheses, one per thread
  if (threadIdx.x < HB) {
    const int t = threadIdx.x;
    uint32_t f = kZeroH;
    if (t < nh) {
      float h[9];
      f = make_hypothesis(a.corr, a.ld, 0, n, a.k0, a.k1, static_cast<uint32_t>(h0 + t), 0u, h);
      score_form(h, a.inv_tau, sm.H[t]);
#pragma unroll
      for (int k = 0; k < 9; ++k) sm.H0[t][k] = h[k];
#pragma unroll
      for (int k = 0; k < 9; ++k) a.hbuf[9ll * (h0 + t) + k] = h[k];
    }
    sm.valid[t] = (t < nh && f == 0u) ? 1u : 0u;
    sm.cnt[t] = 0u;
  }
  if (threadIdx.x == 0) sm.fix.n = 0u;
  __syncthreads();
  // 2. score (validity as a wave-uniform bit mask)
  const int lane = threadIdx.x & 63;
  const uint64_t vmask = __ballot(lane < nh && sm.valid[lane] != 0u);
  score_hyps<P, NW>(a, 0, n, sm.H, vmask, nh, sm.cnt, &sm.fix);
  __syncthreads();
  fix_counts<NW>(a, 0, n, sm.H0, &sm.fix, vmask, nh, sm.cnt, a.hyp_counts != nullptr, sm.ub);
  // 3. publish counts and the block's best key (wave 0 holds all HB <= 64)
  if (threadIdx.x < 64) {
    const int t = threadIdx.x;
    unsigned long long key = 0ull;
    if (t < nh) {
      const uint32_t c = sm.cnt[t];
      const bool ok = sm.valid[t] != 0u;
      if (a.hyp_counts) a.hyp_counts[h0 + t] = ok ? static_cast<int32_t>(c) : 0;
      if (ok) key = pack_key(c, static_cast<uint32_t>(h0 + t));
    }
    key = wave_max_u64(key);
    if (t == 0) a.blockbest[hb] = key;   // reduced by the mask kernel
  }
}

// Persistent (P tiles between checks, HB hypotheses per item): kThreads
// threads, 4 waves per SIMD (128 registers). Single pair (one work item per
// workgroup): kFusedWaves waves, at least 2 per SIMD.
template <int P, int HB, bool PERSISTENT>
__global__ __launch_bounds__(PERSISTENT ? kThreads : kFusedWaves * 64, PERSISTENT ? 4 : 2)
void ransac_kernel(RansacArgs a) {
  if constexpr (!PERSISTENT) {
    __shared__ Smem<HB> sm;
    run_item<P, HB, kFusedWaves>(a, blockIdx.x, sm);
  } else {
    __shared__ TileSmem<HB> sm;
    group_loop<P, HB>(a, sm);
  }
}

// After the persistent kernel (whose keys are then all visible): one workgroup
// per pair writes the pair's best hypothesis, count, index, hypotheses
// evaluated and inlier mask. Fixed count: the pair's key is the atomicMax of
// its blocks' keys. Adaptive termination: the stopping rule applied to the
// published round keys in order, as a sequential loop would (a round before
// the stopping point is always published; if one were missing, n_evaluated
// would read -1).
constexpr int kFinishThreads = 1024;

__global__ __launch_bounds__(kFinishThreads) void ransac_finish_kernel(RansacArgs a) {
  __shared__ float bestH[9];
  __shared__ unsigned long long skey;
  __shared__ int32_t sne;
  const int p = blockIdx.x;
  int64_t base;
  uint32_t n;
  pair_range(a, p, base, n);
  if (a.pst && threadIdx.x < 64) {
    // wave 0: 64 rounds at a time, in order; lane f holds round c0 + f, its
    // prefix maximum (shuffle scan) and whether the rule holds after it
    const int lane = threadIdx.x;
    const uint32_t n_hyp = static_cast<uint32_t>(a.n_hyp);
    const unsigned long long *rk = a.rkey + static_cast<int64_t>(p) * a.n_hb;
    unsigned long long carry = 0ull, key = 0ull;
    int32_t ne = -1;
    for (int c0 = 0; c0 < a.n_hb; c0 += 64) {
      const int f = c0 + lane;
      const unsigned long long k = f < a.n_hb ? rk[f] : kUnpublished;
      const bool pub = k != kUnpublished;
      unsigned long long v = pub ? k : 0ull;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const unsigned long long u = __shfl_up(v, o);
        if (lane >= o) v = max(v, u);
      }
      v = max(v, carry);
      const uint32_t m = min(static_cast<uint32_t>(f + 1) * static_cast<uint32_t>(kRoundHyps),
                             n_hyp);
      const bool stop = f < a.n_hb && pub &&
                        (m >= n_hyp || enough_samples(key_count(v), n, m, a.one_minus_conf));
      const uint64_t sb = __ballot(stop), ub = __ballot(f < a.n_hb && !pub);
      if (sb != 0ull) {
        const int fs = __ffsll(static_cast<long long>(sb)) - 1;   // first round where it holds
        // a round before it unpublished cannot happen (reported as -1)
        const bool gap = (ub & ((2ull << fs) - 1ull)) != 0ull;
        const unsigned long long vk = __shfl(v, fs);
        key = vk;
        ne = gap ? -1 : static_cast<int32_t>(min(static_cast<uint32_t>(c0 + fs + 1) *
                                                     static_cast<uint32_t>(kRoundHyps),
                                                 n_hyp));
        break;
      }
      if (ub != 0ull) break;   // unpublished before any stop: -1
      carry = __shfl(v, 63);
    }
    if (lane == 0) {
      skey = key;
      sne = ne;
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long key;
    int32_t ne;
    if (a.pst) {
      key = skey;
      ne = sne;
    } else {
      key = a.keys[p];
      ne = a.n_hyp;
    }
    if (a.n_eval) a.n_eval[p] = ne;
    if (key != 0ull) {
      const uint32_t hyp = 0xFFFFFFFFu - static_cast<uint32_t>(key & 0xFFFFFFFFull);
      // the winner is recomputed (same device function, same bits) rather than read
      // from another workgroup's memory
      make_hypothesis(a.corr, a.ld, base, n, a.k0, a.k1, hyp, static_cast<uint32_t>(p), bestH);
      a.best_count[p] = static_cast<int32_t>(key_count(key));
      a.best_hyp[p] = static_cast<int32_t>(hyp);
    } else {
#pragma unroll
      for (int k = 0; k < 9; ++k) bestH[k] = 0.0f;
      a.best_count[p] = 0;
      a.best_hyp[p] = -1;
    }
    skey = key;
  }
  __syncthreads();
  if (threadIdx.x < 9) a.best_H[9 * p + threadIdx.x] = bestH[threadIdx.x];
  const bool any = skey != 0ull;
  double hh[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) hh[k] = bestH[k];
  const float *X1 = a.corr + base, *Y1 = a.corr + a.ld + base;
  const float *X2 = a.corr + 2 * a.ld + base, *Y2 = a.corr + 3 * a.ld + base;
  // 4 points per thread in flight (indices clamped into the pair for the loads)
  for (uint32_t i0 = threadIdx.x; i0 < n; i0 += 4u * kFinishThreads) {
    float x1[4], y1[4], x2[4], y2[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const uint32_t j = min(i0 + static_cast<uint32_t>(u) * kFinishThreads, n - 1u);
      x1[u] = X1[j];
      y1[u] = Y1[j];
      x2[u] = X2[j];
      y2[u] = Y2[j];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const uint32_t i = i0 + static_cast<uint32_t>(u) * kFinishThreads;
      if (i < n)
        a.mask[base + i] = (any && inlier_f64(hh, x1[u], y1[u], x2[u], y2[u], a.tau)) ? 1 : 0;
    }
  }
}

// Single pair, after the fused kernel: reduce the work items' best keys (every
// workgroup does it redundantly), then write the best outputs (workgroup 0)
// and this workgroup's slice of the inlier mask.
__global__ __launch_bounds__(kThreads) void ransac_mask_kernel(RansacArgs a) {
  __shared__ unsigned long long red[kWaves];
  __shared__ float bh[9];
  unsigned long long best = 0ull;
  for (int64_t j = threadIdx.x; j < a.n_items; j += kThreads) best = max(best, a.blockbest[j]);
  best = wave_max_u64(best);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = best;
  __syncthreads();
  unsigned long long key = 0ull;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) key = max(key, red[w]);
  const bool any = key != 0ull;
  const uint32_t hyp = any ? 0xFFFFFFFFu - static_cast<uint32_t>(key & 0xFFFFFFFFull) : 0u;
  if (threadIdx.x < 9) bh[threadIdx.x] = any ? a.hbuf[9ull * hyp + threadIdx.x] : 0.0f;
  __syncthreads();
  if (blockIdx.x == 0 && threadIdx.x < 9) a.best_H[threadIdx.x] = bh[threadIdx.x];
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    a.best_count[0] = any ? static_cast<int32_t>((key >> 32) - 1ull) : 0;
    a.best_hyp[0] = any ? static_cast<int32_t>(hyp) : -1;
  }
  double hh[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) hh[k] = bh[k];
  const int n = a.n_single;
  const float *X1 = a.corr, *Y1 = a.corr + a.ld, *X2 = a.corr + 2 * a.ld, *Y2 = a.corr + 3 * a.ld;
  for (int i = blockIdx.x * kThreads + threadIdx.x; i < n; i += gridDim.x * kThreads)
    a.mask[i] = (any && inlier_f64(hh, X1[i], Y1[i], X2[i], Y2[i], a.tau)) ? 1 : 0;
}

// The extent of a pair's points, by pair_waves waves per pair (1 or kWaves).
__device__ void pair_extent(const RansacArgs &a, int block, int pair_waves) {
  __shared__ float part[kWaves][8];
  const int wave = threadIdx.x >> 6;
  const bool solo = pair_waves == 1;
  const int p = solo ? block * kWaves + wave : block;
  int64_t base = 0;
  uint32_t n = 0u;
  if (p < a.n_pairs) pair_range(a, p, base, n);
  const float *X[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) X[k] = a.corr + k * a.ld + base;
  // maxima of x1, y1, x2, y2, then of their negatives
  float m[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) m[k] = -__builtin_inff();
  const uint32_t step = solo ? 64u : kThreads;
  constexpr int kAhead = 8;   // points per thread whose loads are in flight together
  for (uint64_t i0 = solo ? threadIdx.x & 63u : threadIdx.x; i0 < n; i0 += kAhead * step) {
    float v[kAhead][4];
#pragma unroll
    for (int j = 0; j < kAhead; ++j) {
      const uint64_t i = min(i0 + static_cast<uint64_t>(j) * step, static_cast<uint64_t>(n - 1u));
#pragma unroll
      for (int k = 0; k < 4; ++k) v[j][k] = X[k][i];
    }
#pragma unroll
    for (int j = 0; j < kAhead; ++j) {
      if (finite_f(v[j][0]) && finite_f(v[j][1]) && finite_f(v[j][2]) && finite_f(v[j][3])) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          m[k] = fmaxf(m[k], v[j][k]);
          m[4 + k] = fmaxf(m[4 + k], -v[j][k]);
        }
      }
    }
  }
#pragma unroll
  for (int k = 0; k < 8; ++k) m[k] = wave_max_f32(m[k]);
  if (!solo) {
    if ((threadIdx.x & 63) == 0)
#pragma unroll
      for (int k = 0; k < 8; ++k) part[wave][k] = m[k];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 8; ++k)
#pragma unroll
      for (int w = 0; w < kWaves; ++w) m[k] = fmaxf(m[k], part[w][k]);
  }
  const bool writer = solo ? (threadIdx.x & 63) == 0 : threadIdx.x == 0;
  if (!writer || p >= a.n_pairs) return;
  constexpr float up = 1.0f + 9.5367432e-07f;   // above the rounding of the lines below
  Extent x;
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const bool none = !(m[0] > -__builtin_inff());
    const float hi1 = none ? 0.0f : m[k], lo1 = none ? 0.0f : -m[4 + k];
    const float hi2 = none ? 0.0f : m[2 + k], lo2 = none ? 0.0f : -m[6 + k];
    x.c1[k] = 0.5f * lo1 + 0.5f * hi1;
    x.k2[k] = (0.5f * lo2 + 0.5f * hi2) * a.inv_tau;
    x.r1[k] = fmaxf(hi1 - x.c1[k], x.c1[k] - lo1) * up;
    x.r2[k] = fmaxf(fmaf(hi2, a.inv_tau, -x.k2[k]), fmaf(-lo2, a.inv_tau, x.k2[k])) * up;
  }
  a.extent[p] = x;
}

// Resets keys, the queue and the adaptive state, and ranks pairs by size (largest
// first, ties by index). Pair q's sort key is (N_q << 32) | ~q, unique per
// pair, so the rank of p (the number of larger keys) is a permutation of
// 0 .. n_pairs - 1. One wave ranks one pair; the keys are staged through LDS
// in tiles of kThreads, shared by the workgroup's waves. Launched with one
// wave per pair (at least one workgroup); the workgroups past n_prep take the
// pairs' coordinate extents.
__global__ __launch_bounds__(kThreads) void ransac_prep_kernel(RansacArgs a, int rank, int n_prep,
                                                               int pair_waves) {
  __shared__ unsigned long long tile[kThreads];
  if (static_cast<int>(blockIdx.x) >= n_prep) {
    pair_extent(a, static_cast<int>(blockIdx.x) - n_prep, pair_waves);
    return;
  }
  const int64_t g = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  const int64_t stride = static_cast<int64_t>(n_prep) * blockDim.x;
  if (g == 0 && a.queue) *a.queue = 0u;
  for (int64_t q = g; q < a.n_pairs; q += stride) {
    if (a.keys) a.keys[q] = 0ull;
    if (a.pst) {
      a.pst[q].prefix = 0ull;
      a.pst[q].stop = static_cast<uint32_t>(a.n_hb);
      a.pst[q].pad = 0u;
    }
  }
  if (a.rkey) {
    const int64_t total = static_cast<int64_t>(a.n_pairs) * a.n_hb;
    for (int64_t i = g; i < total; i += stride) a.rkey[i] = kUnpublished;
  }
  if (!a.order) return;
  int32_t *order = const_cast<int32_t *>(a.order);
  if (!rank) {
    for (int64_t q = g; q < a.n_pairs; q += stride) order[q] = static_cast<int32_t>(q);
    return;
  }
  auto sort_key = [&](int q) {
    int64_t b;
    uint32_t n = 0u;
    pair_range(a, q, b, n);
    return (static_cast<unsigned long long>(n) << 32) | (0xFFFFFFFFu - static_cast<uint32_t>(q));
  };
  const int p = static_cast<int>(g >> 6);   // this wave's pair (uniform across the wave)
  const int lane = threadIdx.x & 63;
  const unsigned long long kp = p < a.n_pairs ? sort_key(p) : ~0ull;
  int r = 0;
  for (int q0 = 0; q0 < a.n_pairs; q0 += kThreads) {
    const int q = q0 + threadIdx.x;
    __syncthreads();
    tile[threadIdx.x] = q < a.n_pairs ? sort_key(q) : 0ull;   // 0: below every real key
    __syncthreads();
    for (int k = lane; k < kThreads; k += 64) r += tile[k] > kp ? 1 : 0;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) r += __shfl_xor(r, o);
  if (p < a.n_pairs && lane == 0) order[r] = p;
}

// Queue order of the adaptive rounds. Round r of pair p is placed by
// (2r + 1) / N_p, the midpoint of that round on a clock where each of the
// pair's rounds takes N_p units (ties: lower pair index first). The rounds of
// a large pair are spread over the queue instead of being stacked at its end,
// so that the last items are rounds of small pairs; rounds of small pairs
// come later than under plain round order, when more stopping points are
// known. One wave per item: its position is the number of items placed before
// it, counted exactly in integers over all pairs.
__global__ __launch_bounds__(kThreads) void ransac_round_order_kernel(RansacArgs a) {
  __shared__ int64_t nsz[kThreads];
  const int64_t item = (static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x) >> 6;
  const int lane = threadIdx.x & 63;
  const int64_t total = static_cast<int64_t>(a.n_pairs) * a.n_hb;
  const bool live = item < total;   // uniform across the wave
  const int p = live ? static_cast<int>(item / a.n_hb) : 0;
  const int64_t r = live ? item % a.n_hb : 0;
  int64_t b;
  uint32_t n;
  pair_range(a, p, b, n);
  const int64_t np = max(n, 1u);
  const double inv = 1.0 / static_cast<double>(np);
  const int64_t R = a.n_hb;
  const int64_t cap = (2 * R + 2) * np;   // x >= cap: every round of q comes first
  int64_t pos = 0;
  // pair sizes staged through LDS, kThreads at a time, shared by the workgroup's waves
  for (int q0 = 0; q0 < a.n_pairs; q0 += kThreads) {
    __syncthreads();
    if (q0 + static_cast<int>(threadIdx.x) < a.n_pairs) {
      pair_range(a, q0 + threadIdx.x, b, n);
      nsz[threadIdx.x] = max(n, 1u);
    }
    __syncthreads();
    const int qn = min(kThreads, a.n_pairs - q0);
    for (int k = lane; k < qn; k += 64) {
      const int64_t x = (2 * r + 1) * nsz[k];
      if (x >= cap) {
        pos += R;
        continue;
      }
      // c = ceil(x / np): the double estimate is within one of it (x / np < 2R + 2),
      // and one exact integer step corrects it
      int64_t c = static_cast<int64_t>(ceil(static_cast<double>(x) * inv));
      if ((c - 1) * np >= x)
        --c;
      else if (c * np < x)
        ++c;
      // rounds r' of pair q with (2r' + 1) / N_q < (2r + 1) / N_p: the odd numbers below x / np
      pos += min(R, c / 2);
      // equal position: the round (c - 1) / 2 of a lower-numbered pair goes first
      if (q0 + k < p && c * np == x && (c & 1) && (c - 1) / 2 < R) pos += 1;
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) pos += __shfl_xor(pos, o);
  if (live && lane == 0 && pos >= 0 && pos < total)
    a.iorder[pos] = static_cast<int32_t>(static_cast<int64_t>(p) * a.n_hb + r);
}

// ---- plain single-pair form -------------------------------------------------

__global__ void plain_solve_kernel(RansacArgs a, float *Hbuf, uint32_t *valid) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= a.n_hyp) return;
  float h[9];
  const uint32_t f = make_hypothesis(a.corr, a.ld, 0, static_cast<uint32_t>(a.n_single), a.k0,
                                     a.k1, static_cast<uint32_t>(j), 0u, h);
#pragma unroll
  for (int k = 0; k < 9; ++k) Hbuf[9 * j + k] = h[k];
  valid[j] = f == 0u ? 1u : 0u;
}

template <int P, int HB>
__global__ __launch_bounds__(kThreads) void plain_score_kernel(RansacArgs a, const float *Hbuf,
                                                               const uint32_t *valid,
                                                               int32_t *counts) {
  __shared__ float Hs[HB][9];
  __shared__ double H0s[HB][9];
  __shared__ uint32_t vs[HB];
  __shared__ uint32_t cnt[HB];
  __shared__ FixList fix;
  __shared__ uint32_t ub[HB];
  const int h0 = blockIdx.x * HB;
  const int nh = min(HB, a.n_hyp - h0);
  for (int i = threadIdx.x; i < HB * 9; i += kThreads) {
    const float v = (i / 9 < nh) ? Hbuf[9 * h0 + i] : 0.0f;
    Hs[i / 9][i % 9] = (i % 9 < 6) ? v * a.inv_tau : v;   // scoring form
    H0s[i / 9][i % 9] = v;
  }
  for (int i = threadIdx.x; i < HB; i += kThreads) {
    vs[i] = (i < nh) ? valid[h0 + i] : 0u;
    cnt[i] = 0u;
  }
  if (threadIdx.x == 0) fix.n = 0u;
  __syncthreads();
  const int lane = threadIdx.x & 63;
  const uint64_t vmask = __ballot(lane < nh && vs[lane] != 0u);
  score_hyps<P>(a, 0, static_cast<uint32_t>(a.n_single), Hs, vmask, nh, cnt, &fix);
  __syncthreads();
  fix_counts<kWaves>(a, 0, static_cast<uint32_t>(a.n_single), H0s, &fix, vmask, nh, cnt,
             a.hyp_counts != nullptr, ub);
  if (threadIdx.x < nh)
    counts[h0 + threadIdx.x] = vs[threadIdx.x] ? static_cast<int32_t>(cnt[threadIdx.x]) : -1;
}

// One workgroup: argmax over counts (-1 = invalid), ties to the lower index.
constexpr int kArgmaxThreads = 1024;
__global__ __launch_bounds__(kArgmaxThreads) void plain_argmax_kernel(const int32_t *counts,
                                                                      int n_hyp,
                                                                      unsigned long long *key,
                                                                      int32_t *hyp_counts) {
  __shared__ unsigned long long red[kArgmaxThreads / 64];
  unsigned long long best = 0ull;
  for (int j = threadIdx.x; j < n_hyp; j += kArgmaxThreads) {
    const int32_t c = counts[j];
    if (hyp_counts) hyp_counts[j] = c < 0 ? 0 : c;
    if (c >= 0) best = max(best, pack_key(static_cast<uint32_t>(c), static_cast<uint32_t>(j)));
  }
  best = wave_max_u64(best);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = best;
  __syncthreads();
  if (threadIdx.x < 64) {
    unsigned long long v = threadIdx.x < kArgmaxThreads / 64 ? red[threadIdx.x] : 0ull;
    v = wave_max_u64(v);
    if (threadIdx.x == 0) *key = v;
  }
}

__global__ __launch_bounds__(kThreads) void plain_mask_kernel(RansacArgs a, const float *Hbuf,
                                                              const unsigned long long *key) {
  const unsigned long long k = *key;
  const bool any = k != 0ull;
  const uint32_t hyp = any ? 0xFFFFFFFFu - static_cast<uint32_t>(k & 0xFFFFFFFFull) : 0u;
  float bh[9];
  double bd[9];
#pragma unroll
  for (int i = 0; i < 9; ++i) {
    bh[i] = any ? Hbuf[9 * hyp + i] : 0.0f;
    bd[i] = bh[i];
  }
  if (blockIdx.x == 0 && threadIdx.x < 9) a.best_H[threadIdx.x] = bh[threadIdx.x];
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    a.best_count[0] = any ? static_cast<int32_t>((k >> 32) - 1ull) : 0;
    a.best_hyp[0] = any ? static_cast<int32_t>(hyp) : -1;
  }
  const int n = a.n_single;
  const float *X1 = a.corr, *Y1 = a.corr + a.ld, *X2 = a.corr + 2 * a.ld, *Y2 = a.corr + 3 * a.ld;
  for (int i = blockIdx.x * kThreads + threadIdx.x; i < n; i += gridDim.x * kThreads)
    a.mask[i] = (any && inlier_f64(bd, X1[i], Y1[i], X2[i], Y2[i], a.tau)) ? 1 : 0;
}

// ---- tuning --------------------------------------------------------------

struct Tune {
  int P, HB, bpc;
};

static bool tune_valid(const hg_ransac_tuning &t) {
  return (t.pts_per_lane == 8 || t.pts_per_lane == 16) &&
         (t.hyps_per_block == 16 || t.hyps_per_block == 32 || t.hyps_per_block == 64) &&
         t.blocks_per_cu >= 1 && t.blocks_per_cu <= 8;
}

static const hg_ransac_tuning kDefaultTune = {8, 64, 4, 0};

typedef void (*KernelFn)(RansacArgs);

static KernelFn pick_fused(int HB) {
  switch (HB) {
    case 4: return ransac_kernel<8, 4, false>;
    case 8: return ransac_kernel<8, 8, false>;
    case 16: return ransac_kernel<8, 16, false>;
    case 32: return ransac_kernel<8, 32, false>;
    default: return ransac_kernel<8, 64, false>;
  }
}

// Hypotheses of a work item: 32 or 64 (a tuning of 16 runs as 32, the height of a
// tile).
static int item_hyps(const hg_ransac_tuning &t) { return t.hyps_per_block == 64 ? 64 : 32; }

static std::mutex g_tune_mu;
static std::map<std::string, hg_ransac_tuning> g_tune_cache;
static bool g_tune_file_read = false;

static std::string tune_key(int n_pairs, int n_hyp) {
  int dev = 0;
  (void)hipGetDevice(&dev);
  char buf[128];
  snprintf(buf, sizeof buf, "gfx950:%d:%d:%d", device_cus(), n_pairs, n_hyp);
  return buf;
}

static void read_tune_file() {
  if (g_tune_file_read) return;
  g_tune_file_read = true;
  const char *path = getenv("HG_AUTOTUNE_CACHE");
  if (!path) return;
  FILE *f = fopen(path, "r");
  if (!f) return;
  char line[512];
  while (fgets(line, sizeof line, f)) {
    char key[256];
    hg_ransac_tuning t = {0, 0, 0, 0};
    if (sscanf(line, " \"%255[^\"]\" : [ %d , %d , %d ]", key, &t.pts_per_lane,
               &t.hyps_per_block, &t.blocks_per_cu) == 4 &&
        tune_valid(t))
      g_tune_cache[key] = t;
  }
  fclose(f);
}

static void write_tune_file() {
  const char *path = getenv("HG_AUTOTUNE_CACHE");
  if (!path) return;
  FILE *f = fopen(path, "w");
  if (!f) return;
  fprintf(f, "{\n");
  size_t i = 0;
  for (const auto &kv : g_tune_cache) {
    fprintf(f, "  \"%s\": [%d, %d, %d]%s\n", kv.first.c_str(), kv.second.pts_per_lane,
            kv.second.hyps_per_block, kv.second.blocks_per_cu,
            ++i < g_tune_cache.size() ? "," : "");
  }
  fprintf(f, "}\n");
  fclose(f);
}

// The shape of a launch without an explicit tuning: the tuned one of this
// problem, or the default with items of 64 hypotheses, halved where they would be
// fewer than three to each resident workgroup and the pairs are large enough for
// that to matter (64 pairs of up to 8000 points x 1024 hypotheses: 121 us with
// 32, 135 us with 64; 512 pairs: 574 and 563 us; 64 pairs of up to 1000 points:
// 61 and 60 us; 512 of up to 1000: 232 and 185 us). The offsets are on the device, so
// the plane stride stands for the number of points: a slice of longer planes gets
// the shape of larger pairs (its speed alone depends on that).
static hg_ransac_tuning lookup_tune(int n_pairs, int n_hyp, int64_t points) {
  std::lock_guard<std::mutex> lock(g_tune_mu);
  read_tune_file();
  auto it = g_tune_cache.find(tune_key(n_pairs, n_hyp));
  if (it != g_tune_cache.end()) return it->second;
  hg_ransac_tuning t = kDefaultTune;
  const int64_t items = static_cast<int64_t>(n_pairs) * ((n_hyp + 63) / 64);
  const bool large = points / n_pairs >= 1024;
  if (items < (large ? 3072 : 512)) t.hyps_per_block = 32;
  return t;
}

// ---- workspace layout ------------------------------------------------------

static size_t align256(size_t x) { return (x + 255) & ~static_cast<size_t>(255); }

struct BatchedWs {
  unsigned long long *keys;
  int32_t *order;
  uint32_t *queue;
  Extent *extent;
};

static size_t batched_ws_bytes(int n_pairs) {
  return align256(8ull * n_pairs) + align256(4ull * n_pairs) + 256 +
         align256(sizeof(Extent) * static_cast<size_t>(n_pairs));
}

static BatchedWs carve_batched(void *ws, int n_pairs) {
  char *p = static_cast<char *>(ws);
  BatchedWs w;
  w.keys = reinterpret_cast<unsigned long long *>(p);
  p += align256(8ull * n_pairs);
  w.order = reinterpret_cast<int32_t *>(p);
  p += align256(4ull * n_pairs);
  w.queue = reinterpret_cast<uint32_t *>(p);
  p += 256;
  w.extent = reinterpret_cast<Extent *>(p);
  return w;
}

static size_t plain_ws_bytes(int n_hyp) {
  return align256(36ull * n_hyp) + align256(4ull * n_hyp) + align256(4ull * n_hyp) + 256;
}

// ---- host launchers --------------------------------------------------------

static int check_single(const float *corr, int32_t n_pts, int64_t ld, int32_t n_hyp, float thresh,
                        float *best_H, int32_t *best_count, int32_t *best_hyp, uint8_t *mask,
                        void *ws, size_t ws_bytes, size_t need) {
  HG_REQUIRE(corr && best_H && best_count && best_hyp && mask,
             "hg_ransac: NULL corr or output pointer");
  HG_REQUIRE(n_pts >= 4, "hg_ransac: n_pts = %d < 4", n_pts);
  HG_REQUIRE(ld >= n_pts, "hg_ransac: ld < n_pts");
  HG_REQUIRE(n_hyp >= 1, "hg_ransac: n_hyp = %d < 1", n_hyp);
  HG_REQUIRE(std::isfinite(thresh) && thresh > 0.0f && std::isfinite(1.0f / thresh),
             "hg_ransac: threshold must be finite and > 0 (and 1/threshold finite)");
  if (!ws || ws_bytes < need)
    return fail(HG_EWORKSPACE, "hg_ransac: workspace of %zu bytes needed, %zu given", need,
                ws ? ws_bytes : static_cast<size_t>(0));
  HG_REQUIRE(aligned(ws, 256), "hg_ransac: workspace must be 256-byte aligned");
  return HG_OK;
}

static RansacArgs make_args(const float *corr, int64_t ld, const int64_t *off, int32_t n_single,
                            int32_t n_pairs, int32_t n_hyp, int HB, float thresh, uint64_t seed,
                            float *best_H, int32_t *best_count, int32_t *best_hyp, uint8_t *mask,
                            int32_t *hyp_counts) {
  RansacArgs a;
  a.corr = corr;
  a.ld = ld;
  a.off = off;
  a.n_single = n_single;
  a.n_pairs = n_pairs;
  a.n_hyp = n_hyp;
  a.n_hb = (n_hyp + HB - 1) / HB;
  a.n_items = static_cast<int64_t>(n_pairs) * a.n_hb;
  a.tau = thresh;
  a.inv_tau = 1.0f / thresh;
  a.k0 = static_cast<uint32_t>(seed & 0xFFFFFFFFull);
  a.k1 = static_cast<uint32_t>(seed >> 32);
  a.best_H = best_H;
  a.best_count = best_count;
  a.best_hyp = best_hyp;
  a.mask = mask;
  a.hyp_counts = hyp_counts;
  a.keys = nullptr;
  a.queue = nullptr;
  a.order = nullptr;
  a.hbuf = nullptr;
  a.blockbest = nullptr;
  a.pst = nullptr;
  a.rkey = nullptr;
  a.iorder = nullptr;
  a.extent = nullptr;
  a.n_eval = nullptr;
  a.one_minus_conf = 0.0;
  return a;
}

// Enqueue the batched form (prep, round order, persistent kernel, finish) on
// stream s.
static int launch_batched(const RansacArgs &a0, const hg_ransac_tuning &t, void *ws,
                          hipStream_t s) {
  RansacArgs a = a0;
  const BatchedWs w = carve_batched(ws, a.n_pairs);
  a.keys = w.keys;
  a.queue = w.queue;
  a.order = w.order;
  a.extent = w.extent;
  const int rank = a.n_pairs <= 65536 ? 1 : 0;
  // one wave per pair when ranking (ranks of 65536 pairs: 16384 workgroups)
  const int64_t prep_blocks = rank ? (static_cast<int64_t>(a.n_pairs) + kWaves - 1) / kWaves
                                   : (static_cast<int64_t>(a.n_pairs) + kThreads - 1) / kThreads;
  // the extents: a workgroup per pair, or a wave where the pairs are small (by the
  // plane stride, as in lookup_tune)
  const int pair_waves = a.ld / a.n_pairs >= 512 ? kWaves : 1;
  const int64_t ext_blocks = pair_waves == 1 ? (static_cast<int64_t>(a.n_pairs) + kWaves - 1) / kWaves
                                             : a.n_pairs;
  hipLaunchKernelGGL(ransac_prep_kernel, dim3(static_cast<unsigned>(prep_blocks + ext_blocks)),
                     dim3(kThreads), 0, s, a, rank, static_cast<int>(prep_blocks), pair_waves);
  if (int st = launched("ransac_prep_kernel")) return st;
  if (a.iorder) {
    const int64_t waves = static_cast<int64_t>(a.n_pairs) * a.n_hb;
    const int64_t blocks = (waves + kWaves - 1) / kWaves;
    hipLaunchKernelGGL(ransac_round_order_kernel, dim3(static_cast<unsigned>(blocks)),
                       dim3(kThreads), 0, s, a);
    if (int st = launched("ransac_round_order_kernel")) return st;
  }
  const int64_t blocks = std::min<int64_t>(static_cast<int64_t>(device_cus()) * t.blocks_per_cu,
                                           std::max<int64_t>(1, a.n_items));
  const bool deep = t.pts_per_lane != 8;
  auto *k = t.hyps_per_block == 64 ? (deep ? ransac_kernel<32, 64, true> : ransac_kernel<16, 64, true>)
                                   : (deep ? ransac_kernel<32, 32, true> : ransac_kernel<16, 32, true>);
  hipLaunchKernelGGL(k, dim3(static_cast<unsigned>(blocks)), dim3(kThreads), 0, s, a);
  if (int st = launched("ransac_kernel<persistent>")) return st;
  hipLaunchKernelGGL(ransac_finish_kernel, dim3(static_cast<unsigned>(a.n_pairs)),
                     dim3(kFinishThreads), 0, s, a);
  return launched("ransac_finish_kernel");
}

static int check_batched(const float *corr, int64_t ld, const int64_t *off, int32_t n_pairs,
                         int32_t n_hyp, float thresh, const hg_ransac_tuning *tune, float *best_H,
                         int32_t *best_count, int32_t *best_hyp, uint8_t *mask, void *ws,
                         size_t ws_bytes) {
  HG_REQUIRE(corr && off && best_H && best_count && best_hyp && mask,
             "hg_ransac_batched: NULL corr, off or output pointer");
  HG_REQUIRE(n_pairs >= 1, "hg_ransac_batched: n_pairs = %d < 1", n_pairs);
  HG_REQUIRE(ld >= 1, "hg_ransac_batched: ld < 1");
  HG_REQUIRE(n_hyp >= 1, "hg_ransac_batched: n_hyp = %d < 1", n_hyp);
  // the persistent queue is a 32-bit counter that every workgroup also bumps
  // once past the end: at most 2^31 work items (of >= 16 hypotheses) keep it
  // from wrapping, which would restart the queue and never end the launch
  HG_REQUIRE(static_cast<int64_t>(n_pairs) * ((static_cast<int64_t>(n_hyp) + 15) / 16) <=
                 (int64_t(1) << 31),
             "hg_ransac_batched: n_pairs x n_hyp too large for one launch (n_pairs * "
             "ceil(n_hyp / 16) must be <= 2^31)");
  HG_REQUIRE(std::isfinite(thresh) && thresh > 0.0f && std::isfinite(1.0f / thresh),
             "hg_ransac_batched: threshold must be finite and > 0 (and 1/threshold finite)");
  HG_REQUIRE(!tune || tune_valid(*tune), "hg_ransac_batched: unsupported tuning");
  const size_t need = batched_ws_bytes(n_pairs);
  if (!ws || ws_bytes < need)
    return fail(HG_EWORKSPACE, "hg_ransac_batched: workspace of %zu bytes needed, %zu given",
                need, ws ? ws_bytes : static_cast<size_t>(0));
  HG_REQUIRE(aligned(ws, 256), "hg_ransac_batched: workspace must be 256-byte aligned");
  return HG_OK;
}

}  // namespace hg

using namespace hg;

namespace hg {

// Workspace of the fused single-pair form: every hypothesis's H and each work
// item's best key (at least 4 hypotheses per item).
static size_t fused_ws_bytes(int32_t n_hyp) {
  return align256(36ull * n_hyp) + align256(8ull * ((n_hyp + 3) / 4));
}

// Enqueue the fused single-pair form (scoring kernel + mask kernel) with
// workspace ws (validated by the caller).
static int launch_fused(const float *corr, int32_t n_pts, int64_t ld, int32_t n_hyp, float thresh,
                        uint64_t seed, float *best_H, int32_t *best_count, int32_t *best_hyp,
                        uint8_t *inlier_mask, int32_t *hyp_counts, void *ws, hipStream_t s) {
  // about two workgroups per compute unit when the hypothesis count allows it
  int HB = 4;
  while (HB < 64 && static_cast<int64_t>(HB) * 2 * device_cus() < n_hyp) HB *= 2;
  RansacArgs a = make_args(corr, ld, nullptr, n_pts, 1, n_hyp, HB, thresh, seed, best_H,
                           best_count, best_hyp, inlier_mask, hyp_counts);
  char *w = static_cast<char *>(ws);
  a.hbuf = reinterpret_cast<float *>(w);
  a.blockbest = reinterpret_cast<unsigned long long *>(w + align256(36ull * n_hyp));
  KernelFn k = pick_fused(HB);
  hipLaunchKernelGGL(k, dim3(static_cast<unsigned>(a.n_items)), dim3(kFusedWaves * 64), 0, s, a);
  if (int st = launched("ransac_kernel<fused>")) return st;
  const int mb = std::max(1, std::min(1024, (n_pts + kThreads - 1) / kThreads));
  hipLaunchKernelGGL(ransac_mask_kernel, dim3(mb), dim3(kThreads), 0, s, a);
  return launched("ransac_mask_kernel");
}

// The library's own workspace for hg_ransac_noalloc: a static device array
// (each GPU the library runs on holds its own copy until the process ends).
// Host code never uses this name as an address: the device address is looked
// up once per device (hipGetSymbolAddress) and kept in g_noalloc_ws.
constexpr int32_t kNoAllocMaxHyp = 16384;
constexpr size_t kNoAllocBytes = 36ull * kNoAllocMaxHyp + 8ull * (kNoAllocMaxHyp / 4);
static_assert(kNoAllocBytes % 256 == 0, "whole 256-byte blocks");
static __device__ __align__(256) unsigned char scratch[kNoAllocBytes];

static std::mutex g_noalloc_mu;
static void *g_noalloc_ws[64] = {nullptr};

// Device address of `scratch` on the current device (looked up on the first
// call on each device, with that device current).
static int noalloc_ws(void **out) {
  int dev = 0;
  HG_HIP(hipGetDevice(&dev));
  HG_REQUIRE(dev >= 0 && dev < 64, "hg_ransac_noalloc: device ordinal %d out of range", dev);
  std::lock_guard<std::mutex> lock(g_noalloc_mu);
  if (!g_noalloc_ws[dev]) {
    void *ptr = nullptr;
    HG_HIP(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
    HG_REQUIRE(ptr != nullptr && aligned(ptr, 256), "hg_ransac_noalloc: bad workspace address");
    g_noalloc_ws[dev] = ptr;
  }
  *out = g_noalloc_ws[dev];
  return HG_OK;
}

}  // namespace hg

extern "C" size_t hg_ransac_ws_bytes(int32_t n_pts, int32_t n_hyp) {
  (void)n_pts;
  if (n_hyp < 1) n_hyp = 1;
  // fused: H of every hypothesis and per-item best keys; plain: H buffer,
  // validity, counts and the argmax key
  return std::max(fused_ws_bytes(n_hyp), plain_ws_bytes(n_hyp));
}

extern "C" int hg_ransac(const float *corr, int32_t n_pts, int64_t ld, int32_t n_hyp,
                         float thresh, uint64_t seed, float *best_H, int32_t *best_count,
                         int32_t *best_hyp, uint8_t *inlier_mask, int32_t *hyp_counts, void *ws,
                         size_t ws_bytes, void *stream) {
  clear_error();
  if (int st = check_single(corr, n_pts, ld, n_hyp, thresh, best_H, best_count, best_hyp,
                            inlier_mask, ws, ws_bytes, hg_ransac_ws_bytes(n_pts, n_hyp)))
    return st;
  return launch_fused(corr, n_pts, ld, n_hyp, thresh, seed, best_H, best_count, best_hyp,
                      inlier_mask, hyp_counts, ws, as_stream(stream));
}

extern "C" int hg_ransac_noalloc(const float *corr, int32_t n_pts, int64_t ld, int32_t n_hyp,
                                 float thresh, uint64_t seed, float *best_H, int32_t *best_count,
                                 int32_t *best_hyp, uint8_t *inlier_mask, int32_t *hyp_counts,
                                 void *stream) {
  clear_error();
  HG_REQUIRE(n_hyp <= kNoAllocMaxHyp,
             "hg_ransac_noalloc: n_hyp = %d exceeds the maximum of %d (use hg_ransac with a "
             "caller workspace)", n_hyp, kNoAllocMaxHyp);
  // arguments first (host only; any aligned non-null address stands for the
  // workspace here), then the workspace's device address
  if (int st = check_single(corr, n_pts, ld, n_hyp, thresh, best_H, best_count, best_hyp,
                            inlier_mask, reinterpret_cast<void *>(256), kNoAllocBytes,
                            fused_ws_bytes(n_hyp)))
    return st;
  void *ws = nullptr;
  if (int st = noalloc_ws(&ws)) return st;
  return launch_fused(corr, n_pts, ld, n_hyp, thresh, seed, best_H, best_count, best_hyp,
                      inlier_mask, hyp_counts, ws, as_stream(stream));
}

extern "C" int hg_ransac_plain(const float *corr, int32_t n_pts, int64_t ld, int32_t n_hyp,
                               float thresh, uint64_t seed, float *best_H, int32_t *best_count,
                               int32_t *best_hyp, uint8_t *inlier_mask, int32_t *hyp_counts,
                               void *ws, size_t ws_bytes, void *stream) {
  clear_error();
  if (int st = check_single(corr, n_pts, ld, n_hyp, thresh, best_H, best_count, best_hyp,
                            inlier_mask, ws, ws_bytes, hg_ransac_ws_bytes(n_pts, n_hyp)))
    return st;
  const hipStream_t s = as_stream(stream);
  constexpr int HB = 16, P = 8;
  RansacArgs a = make_args(corr, ld, nullptr, n_pts, 1, n_hyp, HB, thresh, seed, best_H,
                           best_count, best_hyp, inlier_mask, hyp_counts);
  char *p = static_cast<char *>(ws);
  float *Hbuf = reinterpret_cast<float *>(p);
  p += align256(36ull * n_hyp);
  uint32_t *valid = reinterpret_cast<uint32_t *>(p);
  p += align256(4ull * n_hyp);
  int32_t *counts = reinterpret_cast<int32_t *>(p);
  p += align256(4ull * n_hyp);
  unsigned long long *key = reinterpret_cast<unsigned long long *>(p);
  hipLaunchKernelGGL(plain_solve_kernel, dim3((n_hyp + 255) / 256), dim3(256), 0, s, a, Hbuf,
                     valid);
  if (int st = launched("plain_solve_kernel")) return st;
  hipLaunchKernelGGL((plain_score_kernel<P, HB>), dim3((n_hyp + HB - 1) / HB), dim3(kThreads), 0,
                     s, a, Hbuf, valid, counts);
  if (int st = launched("plain_score_kernel")) return st;
  hipLaunchKernelGGL(plain_argmax_kernel, dim3(1), dim3(kArgmaxThreads), 0, s, counts, n_hyp, key,
                     hyp_counts);
  if (int st = launched("plain_argmax_kernel")) return st;
  const int mb = std::max(1, std::min(1024, (n_pts + kThreads - 1) / kThreads));
  hipLaunchKernelGGL(plain_mask_kernel, dim3(mb), dim3(kThreads), 0, s, a, Hbuf, key);
  return launched("plain_mask_kernel");
}

extern "C" size_t hg_ransac_batched_ws_bytes(int32_t n_pairs, int32_t n_hyp) {
  (void)n_hyp;
  return batched_ws_bytes(n_pairs < 1 ? 1 : n_pairs);
}

extern "C" int hg_ransac_batched(const float *corr, int64_t ld, const int64_t *off,
                                 int32_t n_pairs, int32_t n_hyp, float thresh, uint64_t seed,
                                 const hg_ransac_tuning *tune, float *best_H, int32_t *best_count,
                                 int32_t *best_hyp, uint8_t *inlier_mask, int32_t *hyp_counts,
                                 void *ws, size_t ws_bytes, void *stream) {
  clear_error();
  if (int st = check_batched(corr, ld, off, n_pairs, n_hyp, thresh, tune, best_H, best_count,
                             best_hyp, inlier_mask, ws, ws_bytes))
    return st;
  const hg_ransac_tuning t = tune ? *tune : lookup_tune(n_pairs, n_hyp, ld);
  RansacArgs a = make_args(corr, ld, off, 0, n_pairs, n_hyp, item_hyps(t), thresh, seed,
                           best_H, best_count, best_hyp, inlier_mask, hyp_counts);
  return launch_batched(a, t, ws, as_stream(stream));
}

extern "C" int hg_ransac_autotune(const float *corr, int64_t ld, const int64_t *off,
                                  const int64_t *off_host, int32_t n_pairs, int32_t n_hyp,
                                  float thresh, uint64_t seed, void *ws, size_t ws_bytes,
                                  void *stream, hg_ransac_tuning *out) {
  clear_error();
  HG_REQUIRE(off_host && out, "hg_ransac_autotune: NULL off_host or out");
  HG_REQUIRE(n_pairs >= 1, "hg_ransac_autotune: n_pairs < 1");
  const int64_t total = off_host[n_pairs];
  HG_REQUIRE(total >= 0 && ld >= total, "hg_ransac_autotune: ld < total points");
  float *bh = nullptr;
  int32_t *bc = nullptr, *bi = nullptr;
  uint8_t *mk = nullptr;
  // validate with dummy output pointers first (host only)
  if (int st = check_batched(corr, ld, off, n_pairs, n_hyp, thresh, nullptr,
                             reinterpret_cast<float *>(1), reinterpret_cast<int32_t *>(1),
                             reinterpret_cast<int32_t *>(1), reinterpret_cast<uint8_t *>(1), ws,
                             ws_bytes))
    return st;
  const hipStream_t s = as_stream(stream);
  hipEvent_t e0 = nullptr, e1 = nullptr;
  // frees whatever was obtained, on every return path
  struct Scratch {
    float **bh;
    int32_t **bc, **bi;
    uint8_t **mk;
    hipEvent_t *e0, *e1;
    ~Scratch() {
      if (*e0) (void)hipEventDestroy(*e0);
      if (*e1) (void)hipEventDestroy(*e1);
      if (*bh) (void)hipFree(*bh);
      if (*bc) (void)hipFree(*bc);
      if (*bi) (void)hipFree(*bi);
      if (*mk) (void)hipFree(*mk);
    }
  } scratch{&bh, &bc, &bi, &mk, &e0, &e1};
  HG_HIP(hipMalloc(&bh, 36ull * n_pairs));
  HG_HIP(hipMalloc(&bc, 4ull * n_pairs));
  HG_HIP(hipMalloc(&bi, 4ull * n_pairs));
  // the kernels clamp pair ranges into [0, ld), so a mask of ld bytes covers any offsets
  HG_HIP(hipMalloc(&mk, static_cast<size_t>(std::max<int64_t>(ld, 1))));
  HG_HIP(hipEventCreate(&e0));
  HG_HIP(hipEventCreate(&e1));
  float best_ms = 1e30f;
  hg_ransac_tuning best = kDefaultTune;
  int status = HG_OK;
  for (int P : {8, 16})
    for (int HB : {32, 64})
      for (int bpc : {1, 2, 4, 5, 6}) {
        const hg_ransac_tuning t = {P, HB, bpc, 0};
        RansacArgs a = make_args(corr, ld, off, 0, n_pairs, n_hyp, item_hyps(t), thresh, seed, bh, bc, bi,
                                 mk, nullptr);
        if ((status = launch_batched(a, t, ws, s)) != HG_OK) goto done;   // warm-up
        float ms[3];
        for (int r = 0; r < 3; ++r) {
          (void)hipEventRecord(e0, s);
          if ((status = launch_batched(a, t, ws, s)) != HG_OK) goto done;
          (void)hipEventRecord(e1, s);
          if (hipEventSynchronize(e1) != hipSuccess) {
            status = fail(HG_EHIP, "autotune: event sync failed");
            goto done;
          }
          (void)hipEventElapsedTime(&ms[r], e0, e1);
        }
        std::sort(ms, ms + 3);
        if (ms[1] < best_ms) {
          best_ms = ms[1];
          best = t;
        }
      }
done:
  (void)hipStreamSynchronize(s);   // the scratch buffers are released when this returns
  if (status != HG_OK) return status;
  *out = best;
  {
    std::lock_guard<std::mutex> lock(g_tune_mu);
    read_tune_file();
    g_tune_cache[tune_key(n_pairs, n_hyp)] = best;
    write_tune_file();
  }
  return HG_OK;
}

// ---- adaptive termination ---------------------------------------------------

constexpr int kRound = kRoundHyps;

static size_t adaptive_extra_bytes(int n_pairs, int n_hyp) {
  const int64_t nr = (static_cast<int64_t>(n_hyp) + kRound - 1) / kRound;
  return align256(sizeof(PairState) * static_cast<size_t>(n_pairs)) +
         align256(8ull * n_pairs * nr) + align256(4ull * n_pairs * nr);
}

// The staggered round order costs n_pairs^2 * rounds integer steps: used up
// to 2^27 of them (e.g. 2048 pairs of 1024 hypotheses), round order beyond.
static bool stagger_rounds(int64_t n_pairs, int64_t n_rounds) {
  return n_pairs * n_pairs * n_rounds <= (int64_t(1) << 27);
}

extern "C" size_t hg_ransac_adaptive_ws_bytes(int32_t n_pairs, int32_t n_hyp_max) {
  if (n_pairs < 1) n_pairs = 1;
  if (n_hyp_max < 1) n_hyp_max = 1;
  return batched_ws_bytes(n_pairs) + adaptive_extra_bytes(n_pairs, n_hyp_max);
}

extern "C" int hg_ransac_adaptive(const float *corr, int64_t ld, const int64_t *off,
                                  int32_t n_pairs, int32_t n_hyp_max, float thresh, uint64_t seed,
                                  double confidence, const hg_ransac_tuning *tune, float *best_H,
                                  int32_t *best_count, int32_t *best_hyp, uint8_t *inlier_mask,
                                  int32_t *n_evaluated, void *ws, size_t ws_bytes, void *stream) {
  clear_error();
  HG_REQUIRE(n_evaluated, "hg_ransac_adaptive: NULL n_evaluated");
  HG_REQUIRE(confidence > 0.0 && confidence < 1.0, "hg_ransac_adaptive: confidence must be in (0, 1)");
  if (int st = check_batched(corr, ld, off, n_pairs, n_hyp_max, thresh, tune, best_H, best_count,
                             best_hyp, inlier_mask, ws, ws_bytes))
    return st;
  const size_t need = hg_ransac_adaptive_ws_bytes(n_pairs, n_hyp_max);
  if (ws_bytes < need)
    return fail(HG_EWORKSPACE, "hg_ransac_adaptive: workspace of %zu bytes needed, %zu given",
                need, ws_bytes);
  hg_ransac_tuning t = tune ? *tune : lookup_tune(n_pairs, n_hyp_max, ld);
  t.hyps_per_block = kRound;   // a work item is one round
  // without an explicit shape: at most 4 workgroups per CU (more rounds in
  // flight at once means more speculative rounds past the stopping points)
  if (!tune) t.blocks_per_cu = std::min(t.blocks_per_cu, 4);
  RansacArgs a = make_args(corr, ld, off, 0, n_pairs, n_hyp_max, kRound, thresh, seed, best_H,
                           best_count, best_hyp, inlier_mask, nullptr);
  char *x = static_cast<char *>(ws) + batched_ws_bytes(n_pairs);
  a.pst = reinterpret_cast<PairState *>(x);
  x += align256(sizeof(PairState) * static_cast<size_t>(n_pairs));
  a.rkey = reinterpret_cast<unsigned long long *>(x);
  x += align256(8ull * n_pairs * a.n_hb);
  if (stagger_rounds(n_pairs, a.n_hb)) a.iorder = reinterpret_cast<int32_t *>(x);
  a.n_eval = n_evaluated;
  a.one_minus_conf = 1.0 - confidence;
  return launch_batched(a, t, ws, as_stream(stream));
}

extern "C" int hg_ransac_batched_graph_create(const float *corr, int64_t ld, const int64_t *off,
                                              int32_t n_pairs, int32_t n_hyp, float thresh,
                                              uint64_t seed, const hg_ransac_tuning *tune,
                                              float *best_H, int32_t *best_count,
                                              int32_t *best_hyp, uint8_t *inlier_mask,
                                              int32_t *hyp_counts, void *ws, size_t ws_bytes,
                                              void *stream, hg_graph **out) {
  clear_error();
  HG_REQUIRE(out, "hg_ransac_batched_graph_create: NULL out");
  *out = nullptr;
  if (int st = check_batched(corr, ld, off, n_pairs, n_hyp, thresh, tune, best_H, best_count,
                             best_hyp, inlier_mask, ws, ws_bytes))
    return st;
  const hg_ransac_tuning t = tune ? *tune : lookup_tune(n_pairs, n_hyp, ld);
  RansacArgs a = make_args(corr, ld, off, 0, n_pairs, n_hyp, item_hyps(t), thresh, seed,
                           best_H, best_count, best_hyp, inlier_mask, hyp_counts);
  return capture_graph(stream, [&](hipStream_t cap) { return launch_batched(a, t, ws, cap); },
                       out);
}

extern "C" int hg_graph_launch(hg_graph *g, void *stream) {
  clear_error();
  HG_REQUIRE(g && g->exec, "hg_graph_launch: NULL graph");
  HG_HIP(hipGraphLaunch(g->exec, as_stream(stream)));
  return HG_OK;
}

extern "C" void hg_graph_destroy(hg_graph *g) {
  if (!g) return;
  if (g->exec) (void)hipGraphExecDestroy(g->exec);
  if (g->graph) (void)hipGraphDestroy(g->graph);
  delete g;
}
