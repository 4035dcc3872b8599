// lyaf_instrument.hip -- the instrument model applied to the transmitted flux
// (Greig, Bolton & Wyithe 2011, Section 3.1 for the high-resolution mock
// spectra, Section 3.2 for the BOSS-like ones, Section 4.2 for the SDSS-like
// ones): convolution with a Gaussian line-spread function, resampling onto
// coarser bins, additive noise.
//
//   Fc_i   = sum_m c_m F_{(i-m) mod N},  c_m = g(m dv) / Z,  g(d) = exp(-(d/b_L)^2),
//            b_L = FWHM / (2 sqrt(ln 2)), m over |m dv| <= k b_L (or the whole
//            box at minimal images), Z = sum_m g(m dv)
//   Fbin_k = average over bin k ([v0 + k dv_bin, v0 + (k+1) dv_bin), periodic)
//            of the piecewise-constant spectrum that takes the value Fc_i on
//            pixel i = [(i - 1/2) dv, (i + 1/2) dv)
//   Fobs_k = Fbin_k + sigma eps_k
//
// Kernel layout.  Line-spread functions whose taps fit one block of kInsTapBlock (all
// but those of several pixels' width) take a wave per part of a skewer, with no
// barrier: it forms the taps once and walks pieces of 512 outputs, eight consecutive
// ones to a lane.  The flux of a piece with its halo of M pixels on each side sits in
// LDS as FP32 in 8 planes by index mod 8 (lane l reads element 8l + j from plane j, so
// the reads of a wave are consecutive); the lane walks the taps with two windows of
// registers used in turn, accumulating in FP64 (on gfx950 an FP64 FMA issues at the
// rate of an unpacked FP32 one).  The convolved span then becomes an FP64 prefix sum
// in LDS, and each bin is the difference of that cumulative integral, linearly
// interpolated, at its two edges, divided by its width.  Wider line-spread functions
// take a workgroup per skewer, which walks tiles of kInsTile pixels and stages FP64
// values and the taps block by block.
//
// The backward is the transpose: each pixel gathers the gradients of the bins it
// overlaps (times overlap / bin width), and the same convolution runs over those
// values (the taps are even in m).  A wave per part again, where the bins over a
// staged piece are few enough: their FP64 prefix sums go to LDS, and a pixel's
// gathered gradient is the difference of their linear interpolation at its two edges.
// Other skewers of at most kInsBwdBins bins (wide line-spread functions, bins finer
// than pixels) take the workgroup, which sums all of the bins; skewers with more bins
// one workgroup per tile, gathering by a merge walk over the bins in memory.
//
// 4096 skewers of 4096 pixels at 2 km/s (FWHM 7, bins of 3.08 km/s; 222 MB moved) and
// at 18.3 km/s (FWHM 224, bins of 64 km/s), forward and backward together: 195 and
// 198 -> 147 and 157 us, where a workgroup per skewer with tiles of 2048 waited at
// five barriers per tile and left a third of its waves without outputs in the last
// one.  Vector issue takes about half of that, the traffic a quarter; the FP64
// windows hold the kernels to four waves per SIMD (at five they spill: 94 against 88
// and 188 against 92 us), which do not hide the rest.
#include <algorithm>

#include "lyaf_internal.h"

namespace lyaf {
namespace {

constexpr int kInsThreads = 256;
constexpr int kInsPerLane = 8;                       // outputs per lane
constexpr int kInsTile = kInsThreads * kInsPerLane;  // 2048 pixels
constexpr int kInsWindow = 1792;                     // bin lower edges per item
constexpr int kInsTapBlock = 256;                    // taps staged at once
// Doubles per plane: at least (tile + tap block) / 8, and 2 * stride = 16 mod
// 64 dwords, so that the 64 lanes of a staging write (8 planes x 8 rows) hit 64
// different bank pairs.
constexpr int kInsPlane = 296;
static_assert(8 * kInsPlane >= kInsTile + kInsTapBlock + 16, "staged block must fit");
static_assert((2 * kInsPlane) % 64 == 16, "planes must start on different banks");
static_assert(kInsMaxRatio + kInsWindow + 4 <= kInsTile, "bin span must fit the tile");
static_assert(kInsTapBlock % 16 == 0, "tap blocks are walked 16 at a time");

// A double that every lane of the wave holds alike, moved to scalar registers:
// FP64 arithmetic runs on the vector unit, so the skewer and tile constants
// would otherwise take a register pair in every lane for the whole walk.
__device__ inline double wave_uniform(double x) {
  const uint64_t b = (uint64_t)__double_as_longlong(x);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)b);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(b >> 32));
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// Per-skewer geometry shared by both kernels.
struct InsSkewer {
  int64_t off, n, out_off, n_out;
  double dv;       // pixel width, km/s
  double inv_dv;   // 1 / dv
  double q;        // bin width in pixels
  double inv_q;    // 1 / q
  int M;           // taps m = -M .. M
  bool half_ends;  // the two extreme taps are the same image (whole even box)
  bool ok;
};

__device__ InsSkewer ins_skewer(const InsArgs &a, int64_t s) {
  InsSkewer k;
  k.off = a.offsets[s];
  k.n = a.offsets[s + 1] - k.off;
  k.out_off = a.out_offsets[s];
  k.n_out = a.out_offsets[s + 1] - k.out_off;
  k.dv = wave_uniform((double)a.dv[s]);
  k.inv_dv = wave_uniform(1.0 / k.dv);
  k.q = wave_uniform(a.bin * k.inv_dv);
  k.inv_q = wave_uniform(k.dv * a.inv_bin);
  k.ok = k.dv > 0.0 && isfinite(k.dv) &&
         (k.n_out == 0 || (k.q <= (double)kInsMaxRatio &&
                           (double)k.n_out * a.bin <= (double)(int)k.n * k.dv * (1.0 + 1e-9)));
  k.M = 0;
  k.half_ends = false;
  if (a.fwhm > 0.0) {
    const double reach = a.window_k * a.fwhm * kInvTwoSqrtLn2 * k.inv_dv;  // k b_L / dv
    if (a.window_k > 0.0 && reach < 0.5 * (double)((int)k.n - 1)) {
      k.M = (int)floor(reach);
    } else {  // the whole box, every offset at its minimal image
      k.M = (int)(k.n / 2);
      k.half_ends = (k.n % 2) == 0;
    }
  }
  return k;
}

// Lower edge of bin k in pixel coordinates (pixel i is [i, i+1)).
__device__ inline double bin_edge(const InsArgs &a, const InsSkewer &k, int64_t bin) {
  return __builtin_fma((double)bin, a.bin, a.v_start) * k.inv_dv + 0.5;
}

// i mod n in [0, n) for |i| < 2^52, 1 <= n <= 2^24 (a skewer's length).
__device__ inline int64_t wrap_index(int64_t i, int n) {
  int64_t r = i - (int64_t)floor((double)i / (double)n) * n;
  if (r < 0) r += n;
  if (r >= n) r -= n;
  return r;
}

// LDS of one workgroup.
struct InsShared {
  double s[8 * kInsPlane];  // staged values in 8 planes, later the prefix sums
  double h[kInsTapBlock];   // taps of the current block
  double red[kInsThreads / 64];
};

__device__ inline void stage_store(InsShared &sh, int x, double v) {
  sh.s[(x & 7) * kInsPlane + (x >> 3)] = v;
}

// Sum over the workgroup, in a fixed order.
__device__ double block_sum_d(double v, double *red) {
  for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  double t = 0.0;
#pragma unroll
  for (int w = 0; w < kInsThreads / 64; ++w) t += red[w];
  return t;
}

// The unnormalised tap at offset m, |m| <= M: g(m dv), halved at the two ends
// of a whole even box; scale = dv / b_L.
__device__ inline double tap_value(const InsArgs &a, const InsSkewer &k, int m, double scale) {
  if (!(a.fwhm > 0.0)) return 1.0;  // M = 0: the identity
  const double x = (double)m * scale;
  double g = exp(-x * x);
  if (k.half_ends && (m == k.M || m == -k.M)) g *= 0.5;
  return g;
}
__device__ inline double tap_scale(const InsArgs &a, const InsSkewer &k) {
  return a.fwhm > 0.0 ? k.dv / (a.fwhm * kInvTwoSqrtLn2) : 0.0;
}

// Taps u0 .. u0 + tbp - 1 of the walk (h_u = g((M - u) dv), zero past the tb
// real ones) into sh.h; returns this thread's share of their sum.
__device__ double stage_taps(const InsArgs &a, const InsSkewer &k, int u0, int tb, int tbp,
                             double *h) {
  double z_part = 0.0;
  const double scale = tap_scale(a, k);
  for (int u = threadIdx.x; u < tbp; u += kInsThreads) {
    const double g = u < tb ? tap_value(a, k, k.M - (u0 + u), scale) : 0.0;
    h[u] = g;
    z_part += g;
  }
  return z_part;
}

// Four taps against the window lo (elements 8l + u .. 8l + u + 7) and hi (the next
// 8), HALF of eight taps: taps u + 4 HALF .. u + 4 HALF + 3 reach elements up to
// 4 HALF + 3 of hi.
template <int HALF>
__device__ __forceinline__ void conv_half(const double (&lo)[8], const double (&hi)[8],
                                          const double (&t)[4], double (&acc)[kInsPerLane]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
#pragma unroll
    for (int q = 0; q < kInsPerLane; ++q) {
      const int e = q + i + 4 * HALF;
      acc[q] = __builtin_fma(t[i], e < 8 ? lo[e] : hi[e - 8], acc[q]);
    }
  }
}

// acc[q] += sum_{u < tbp} h_u s[8l + q + u] over a staged block (tbp a multiple of
// 8): lane l owns outputs 8l .. 8l + 7; element 8l + 8b + j of the block sits in
// plane j at row l + b, p is the lane's row of plane 0 and PLANE the planes' stride.
// Half a window is read ahead of the four taps that need it and no more (the
// schedule is held to that, or the taps' reads take the registers).
template <int PLANE, class E>
__device__ __forceinline__ void conv_walk(int tbp, double (&acc)[kInsPerLane], const E *p,
                                          const double *taps) {
  double wa[8], wb[8];
  E f[4], g[4];
#pragma unroll
  for (int j = 0; j < 8; ++j) wa[j] = (double)p[j * PLANE];
#pragma unroll
  for (int j = 0; j < 4; ++j) f[j] = p[j * PLANE + 1];
  const auto step = [&](int u, const double(&lo)[8], double(&hi)[8]) {
    const E *pb = p + (u >> 3);
    double t[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) t[i] = taps[u + i];
#pragma unroll
    for (int j = 0; j < 4; ++j) g[j] = pb[(4 + j) * PLANE + 1];
#pragma unroll
    for (int j = 0; j < 4; ++j) hi[j] = (double)f[j];
    conv_half<0>(lo, hi, t, acc);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < 4; ++i) t[i] = taps[u + 4 + i];
#pragma unroll
    for (int j = 0; j < 4; ++j) f[j] = pb[j * PLANE + 2];
#pragma unroll
    for (int j = 0; j < 4; ++j) hi[4 + j] = (double)g[j];
    conv_half<1>(lo, hi, t, acc);
    __builtin_amdgcn_sched_barrier(0);
  };
  int u = 0;
  for (; u + 16 <= tbp; u += 16) {
    step(u, wa, wb);
    step(u + 8, wb, wa);
  }
  if (u < tbp) step(u, wa, wb);
}

// Convolution of a tile: acc[q] = sum_{u < T} h_u src(8l + q + u) for the lane's
// outputs t = 8l + q < span, taps in blocks of kInsTapBlock (unnormalised; the
// sum of the taps is returned).  src(x) yields the value at staged offset x
// (x = 0 .. span + T - 2).
template <class Src>
__device__ double convolve_tile(const InsArgs &a, const InsSkewer &k, int span, Src src,
                                double (&acc)[kInsPerLane], InsShared &sh) {
  const int T = 2 * k.M + 1;
  const int tid = threadIdx.x;
  const bool wave_active = (tid & ~63) * kInsPerLane < span;
  double z_part = 0.0;
#pragma unroll
  for (int q = 0; q < kInsPerLane; ++q) acc[q] = 0.0;
  for (int u0 = 0; u0 < T; u0 += kInsTapBlock) {
    const int tb = min(kInsTapBlock, T - u0);  // real taps in this block
    const int tbp = (tb + 15) & ~15;           // walked taps (zero-padded)
    __syncthreads();  // the previous block's readers are done
    z_part += stage_taps(a, k, u0, tb, tbp, sh.h);
    const int need = span + tbp - 1;  // staged offsets read by outputs < span
    const int real = span + tb - 1;   // offsets carrying real taps
    for (int x = tid; x < need; x += kInsThreads) stage_store(sh, x, x < real ? src(u0 + x) : 0.0);
    __syncthreads();
    if (wave_active) conv_walk<kInsPlane>(tbp, acc, sh.s + threadIdx.x, sh.h);
  }
  return block_sum_d(z_part, sh.red);
}

// Geometry of tile c of a skewer: the bins whose lower edge lies in pixels
// [c W, (c+1) W) from the first bin's edge, and the pixels they cover.
struct InsTile {
  int64_t k_lo, k_hi;  // bins k_lo .. k_hi - 1 (none if k_lo >= k_hi)
  int64_t p0;          // first pixel of the span (absolute; may lie outside [0, n))
  double e_lo;         // lower edge of bin k_lo relative to p0, pixels
  double xb;           // lower edge of bin k_hi, pixels
  uint32_t base;       // (p0 - M) mod n: pixel of staged offset 0
  int span;            // pixels covered
};

__device__ inline int64_t first_bin(const InsSkewer &k, int64_t c) {
  if (c == 0) return 0;
  if (c * kInsWindow >= k.n) return k.n_out;  // past the last tile
  // c kInsWindow < n, so kb <= n / q + 1, about n_out + 1: exact as int64
  const int64_t kb = (int64_t)ceil((double)(c * kInsWindow) * k.inv_q);
  return kb >= k.n_out ? k.n_out : kb;
}

// Tile c, given tile c - 1 (prev, for c > 0): the lower bin and edge of a tile
// are the upper ones of the one before, and its base moves with p0.
__device__ InsTile ins_tile(const InsArgs &a, const InsSkewer &k, int c, const InsTile *prev) {
  InsTile t;
  double xa;
  if (prev) {
    t.k_lo = prev->k_hi;
    xa = prev->xb;
  } else {
    t.k_lo = 0;
    xa = bin_edge(a, k, 0);
  }
  t.k_hi = first_bin(k, c + 1);
  t.p0 = 0;
  t.e_lo = 0.0;
  t.xb = xa;
  t.base = 0;
  t.span = 0;
  if (t.k_lo < t.k_hi) {
    t.xb = wave_uniform(bin_edge(a, k, t.k_hi));
    t.p0 = (int64_t)floor(xa);
    t.e_lo = wave_uniform(xa - (double)t.p0);
    t.span = (int)((int64_t)floor(t.xb) - t.p0 + 1);
    const int64_t step = prev ? t.p0 - prev->p0 : 0;  // 0 <= step <= kInsTile
    if (prev && step < k.n) {
      int64_t b = (int64_t)prev->base + step;
      if (b >= k.n) b -= k.n;
      t.base = (uint32_t)b;
    } else {
      t.base = (uint32_t)wrap_index(t.p0 - k.M, (int)k.n);
    }
  }
  return t;
}

// Staged offset x of a tile holds pixel (p0 - M + x) mod n; n <= 2^24, so 32
// bits do.
__device__ inline float tile_flux(const float *F, uint32_t n32, uint32_t base, int x) {
  uint32_t i = base + (uint32_t)x;
  if (i >= n32) i -= n32;
  if (i >= n32) i %= n32;
  return F[i];
}

// Thread t writes the bins j0 .. j0 + cnt - 1 of a tile (consecutive, so that
// neighbouring bins share the cumulative value at their common edge).
__device__ inline void bin_range(const InsTile &t, int &j0, int &cnt) {
  const int nb = (int)(t.k_hi - t.k_lo);
  const int cb = (nb + kInsThreads - 1) / kInsThreads;
  j0 = min((int)threadIdx.x * cb, nb);
  cnt = min(cb, nb - j0);
}

constexpr int kTileRows = 320;  // rows of a plane of a staged FP32 tile, 5 blocks of 64
static_assert(8 * kTileRows >= kInsTile + kInsTapBlock + 16, "a staged tile must fit");

// Prefix sums of a convolved tile, then its bins: each bin is the difference of the
// interpolated cumulative integral at its edges e(j) = e_lo + j q (relative to p0),
// divided by its width.
__device__ void finish_tile(const InsArgs &a, const InsSkewer &k, const InsTile &t,
                            const double (&acc)[kInsPerLane], double Z, double *pre,
                            double *red) {
  const int span = t.span;
  // pre[i] = sum_{i' < i} Fc[i']; only outputs inside the span enter (lanes
  // past it hold garbage)
  const double invZ = 1.0 / Z;
  const int t0 = threadIdx.x * kInsPerLane;
  double run = 0.0, loc[kInsPerLane];
#pragma unroll
  for (int q = 0; q < kInsPerLane; ++q) {
    if (t0 + q < span) run += acc[q] * invZ;
    loc[q] = run;
  }
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  double incl = run;
  for (int d = 1; d < 64; d <<= 1) {
    const double o = __shfl_up(incl, d);
    if (lane >= d) incl += o;
  }
  __syncthreads();  // every wave is done with the staged values
  if (lane == 63) red[wv] = incl;
  __syncthreads();
  double excl = incl - run;
  for (int w = 0; w < wv; ++w) excl += red[w];
  if (threadIdx.x == 0) pre[0] = 0.0;
#pragma unroll
  for (int q = 0; q < kInsPerLane; ++q)
    if (t0 + q < span) pre[t0 + q + 1] = excl + loc[q];
  __syncthreads();

  const auto cum = [&](double e) -> double {
    const int i = min((int)e, span - 1);
    const double f = e - (double)i;
    return __builtin_fma(f, pre[i + 1] - pre[i], pre[i]);
  };
  int j0, cnt;
  bin_range(t, j0, cnt);
  if (cnt <= 0) return;
  float *out = a.out + k.out_off + t.k_lo + j0;
  const float *noise = a.noise ? a.noise + k.out_off + t.k_lo + j0 : nullptr;
  double c0 = cum(__builtin_fma((double)j0, k.q, t.e_lo));
  for (int r = 0; r < cnt; ++r) {
    const double c1 = cum(__builtin_fma((double)(j0 + r + 1), k.q, t.e_lo));
    out[r] = (float)__builtin_fma(c1 - c0, k.inv_q, a.sigma * (double)(noise ? noise[r] : 0.0f));
    c0 = c1;
  }
}

// ---- Line-spread functions of one block of taps: a wave per piece ----
//
// A wave takes kInsPiece outputs, eight to a lane, with their halo, through LDS of
// its own: the staged flux (FP32, 8 planes of kPieceRows rows: element x at plane
// x mod 8, row x / 8; 64 lanes write and read 64 different banks), later the
// prefix sums.  The waves of a workgroup share the skewer's taps and no barrier.
constexpr int kInsPiece = 64 * kInsPerLane;  // 512
constexpr int kInsWaves = kInsThreads / 64;
static_assert(kInsWaves == 4, "a workgroup holds whole skewers of 1, 2 or 4 parts");
constexpr int kPieceRows = 104;
constexpr int kPieceDoubles = 9 * 64;  // prefix sums, nine to a lane
constexpr int kPieceLoads = (kInsPiece + kInsTapBlock) / 64;
static_assert(8 * kPieceRows >= kInsPiece + kInsTapBlock + 16, "a staged piece must fit");
static_assert(kPieceRows % 16 == 8, "planes must start on different banks");
static_assert(8 * kPieceRows * sizeof(float) <= kPieceDoubles * sizeof(double),
              "the prefix sums take the staged values' place");
static_assert(kInsMaxRatio + 3 < kInsPiece / 2 + 1, "half a piece is left at the widest bins");

// LDS operations of a wave complete in order: only the compiler has to keep it.
__device__ __forceinline__ void wave_lds_order() { asm volatile("" ::: "memory"); }

template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_add_d(double x) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), CTRL, ROWS, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), CTRL, ROWS, 0xF, false);
  return x + __hiloint2double(hi, lo);
}
// Inclusive sums over the wave.
__device__ __forceinline__ double wave_scan_d(double x) {
  x = dpp_add_d<0x111, 0xF>(x);  // row_shr:1, 2, 4, 8 (zero from outside the row)
  x = dpp_add_d<0x112, 0xF>(x);
  x = dpp_add_d<0x114, 0xF>(x);
  x = dpp_add_d<0x118, 0xF>(x);
  x = dpp_add_d<0x142, 0xA>(x);  // row_bcast:15 into rows 1 and 3
  x = dpp_add_d<0x143, 0xC>(x);  // row_bcast:31 into rows 2 and 3
  return x;
}
// x of the lane below, 0 in lane 0.
__device__ __forceinline__ double wave_below_d(double x) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), 0x138, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), 0x138, 0xF, 0xF, false);
  return __hiloint2double(hi, lo);  // wave_shr:1
}

// x of the lane above, 0 in lane 63.
__device__ __forceinline__ double wave_above_d(double x) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), 0x130, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), 0x130, 0xF, 0xF, false);
  return __hiloint2double(hi, lo);  // wave_shl:1
}

__device__ inline int64_t uniform_i64(int64_t x) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)(uint64_t)x);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)x >> 32));
  return (int64_t)(((uint64_t)hi << 32) | lo);
}

// i mod n in [0, n) as wrap_index, by the rounded inverse of n (the quotient is
// off by one at most).
__device__ inline uint32_t wrap_fast(double i, double nd, double inv_nd) {
  double r = __builtin_fma(-floor(i * inv_nd), nd, i);
  if (r < 0.0) r += nd;
  if (r >= nd) r -= nd;
  return (uint32_t)r;
}

// The skewer's taps into the wave's h; returns the inverse of their sum.
__device__ __forceinline__ double wave_taps(const InsArgs &a, const InsSkewer &k, double *h) {
  const int T = 2 * k.M + 1, tbp = (T + 7) & ~7;
  const double scale = tap_scale(a, k);
  double z = 0.0;
  wave_lds_order();
  for (int u = threadIdx.x & 63; u < tbp; u += 64) {
    const double g = u < T ? tap_value(a, k, k.M - u, scale) : 0.0;
    h[u] = g;
    z += g;
  }
  wave_lds_order();
  z = wave_scan_d(z);
  const int lo = __builtin_amdgcn_readlane(__double2loint(z), 63);
  const int hi = __builtin_amdgcn_readlane(__double2hiint(z), 63);
  return 1.0 / __hiloint2double(hi, lo);
}

// Piece c of the forward: the bins whose lower edge lies in pixels [c W, (c+1) W)
// from the first bin's edge, W = kInsPiece - 3 - ceil(bin width), so that the
// pixels they cover are at most kInsPiece.
struct InsPiece {
  int64_t k_lo;   // first bin
  int nb;         // bins (none: past the last)
  int span;       // pixels covered
  uint32_t base;  // pixel of staged offset 0
  double e_lo;    // lower edge of the first bin relative to the span, pixels
};
__device__ inline InsPiece ins_piece(const InsArgs &a, const InsSkewer &k, int c, int W, double nd,
                                     double inv_nd) {
  const auto first = [&](int64_t x) -> int64_t {  // first bin from pixel x on
    if (x >= k.n) return k.n_out;
    const int64_t kb = (int64_t)ceil((double)(int)x * k.inv_q);
    return kb >= k.n_out ? k.n_out : kb;
  };
  InsPiece t;
  t.k_lo = uniform_i64(c == 0 ? 0 : first((int64_t)c * W));
  const int64_t k_hi = uniform_i64(first((int64_t)(c + 1) * W));
  t.nb = (int)(k_hi - t.k_lo);
  t.span = 0;
  t.base = 0;
  t.e_lo = 0.0;
  if (t.nb > 0) {
    const double xa = bin_edge(a, k, t.k_lo), xb = bin_edge(a, k, k_hi);
    const double p0 = floor(xa);
    t.e_lo = wave_uniform(xa - p0);
    t.span = __builtin_amdgcn_readfirstlane((int)(floor(xb) - p0) + 1);
    t.base = __builtin_amdgcn_readfirstlane(wrap_fast(p0 - (double)k.M, nd, inv_nd));
  }
  return t;
}

// The forward of one wave: pieces part, part + parts, .. of the skewer, the flux of
// the next one read into registers while this one's bins are formed.
__device__ __forceinline__ void ins_forward_pieces(const InsArgs &a, const InsSkewer &k,
                                                   double *lds, double *taps, int part,
                                                   int parts) {
  const int lane = threadIdx.x & 63;
  const int T = 2 * k.M + 1, tbp = (T + 7) & ~7;
  const int W = __builtin_amdgcn_readfirstlane(kInsPiece - 3 - (int)ceil(k.q));
  const int nt = (int)((k.n + W - 1) / W);
  const double nd = (double)(int)k.n, inv_nd = wave_uniform(1.0 / nd);
  const uint32_t n32 = (uint32_t)k.n;
  const float *F = a.in + k.off;
  float *st = reinterpret_cast<float *>(lds);
  float R[kPieceLoads];
  const auto load = [&](const InsPiece &t) {
    const int real = t.span + T - 1, nr = (t.span + tbp - 1 + 63) >> 6;
    const bool whole = t.base + (uint32_t)real <= n32;  // no end of the box inside
#pragma unroll
    for (int r = 0; r < kPieceLoads; ++r) {
      R[r] = 0.0f;
      if (r < nr) {
        const int x = 64 * r + lane;
        uint32_t i = t.base + (uint32_t)(x < real ? x : 0);
        if (!whole) i = i >= n32 ? (i - n32 >= n32 ? i % n32 : i - n32) : i;
        R[r] = F[i];
      }
    }
  };
  if (part >= nt) return;
  InsPiece t = ins_piece(a, k, part, W, nd, inv_nd);
  if (t.nb > 0 && t.span <= kInsPiece) load(t);
  const double invZ = wave_taps(a, k, taps);  // while the first piece's flux is on its way
  for (int c = part; c < nt && t.nb > 0; c += parts) {
    if (t.span > kInsPiece) {  // excluded by the bin-width limit; never expected
      if (lane == 0) atomicOr(a.status, LYAF_STATUS_DOMAIN);
      return;
    }
    {
      const int real = t.span + T - 1, nr = (t.span + tbp - 1 + 63) >> 6;
      float *w = st + (lane & 7) * kPieceRows + (lane >> 3);
      wave_lds_order();
#pragma unroll
      for (int r = 0; r < kPieceLoads; ++r)
        if (r < nr) w[8 * r] = 64 * r + lane < real ? R[r] : 0.0f;
      wave_lds_order();
    }
    InsPiece tn = t;
    tn.nb = 0;
    if (c + parts < nt) tn = ins_piece(a, k, c + parts, W, nd, inv_nd);
    const float *noise = a.noise ? a.noise + k.out_off + t.k_lo : nullptr;
    double acc[kInsPerLane];
#pragma unroll
    for (int q = 0; q < kInsPerLane; ++q) acc[q] = 0.0;
    conv_walk<kPieceRows>(tbp, acc, st + lane, taps);
    if (tn.nb > 0 && tn.span <= kInsPiece) load(tn);
    // prefix sums: pre[9 l + q] = sum of the outputs before 8 l + q, q = 0 .. 8 (the
    // neighbours of an interpolation are then in one row).  Outputs past the span
    // enter only sums past it.
    double run = 0.0;
#pragma unroll
    for (int q = 0; q < kInsPerLane; ++q) {
      acc[q] *= invZ;
      run += acc[q];
    }
    double s = wave_below_d(wave_scan_d(run));
    wave_lds_order();
    double *pre = lds + 9 * lane;
    pre[0] = s;
#pragma unroll
    for (int q = 0; q < kInsPerLane; ++q) {
      s += acc[q];
      pre[q + 1] = s;
    }
    wave_lds_order();
    const int last = t.span - 1;
    const auto cum = [&](double e) -> double {
      const int i = min((int)e, last);
      const double f = e - (double)i;
      const double *r = lds + (i + (i >> 3));
      return __builtin_fma(f, r[1] - r[0], r[0]);
    };
    float *out = a.out + k.out_off + t.k_lo;
    // 63 bins at a time: a bin's upper edge is the lower one of the lane above
    for (int j0 = 0; j0 < t.nb; j0 += 63) {
      const int j = j0 + lane;
      const float z = noise ? noise[min(j, t.nb - 1)] : 0.0f;
      const double c0 = cum(fmin(__builtin_fma((double)j, k.q, t.e_lo), (double)t.span));
      const double c1 = wave_above_d(c0);
      if (lane < 63 && j < t.nb)
        out[j] = (float)__builtin_fma(c1 - c0, k.inv_q, a.sigma * (double)z);
    }
    t = tn;
  }
}

// Forward.  When the taps fit one block (2M + 1 <= kInsTapBlock) a wave walks a
// skewer, or one of its parts, by itself; wider line-spread functions stage the taps
// block by block for every tile, the workgroup together.
struct InsPieceShared {
  double w[kInsWaves][kPieceDoubles];
  double h[kInsWaves][kInsTapBlock];
};
union InsLds {
  InsShared w;       // wide line-spread functions
  InsPieceShared p;  // taps in one block
};

__device__ void ins_forward_wide(const InsArgs &a, const InsSkewer &k, InsShared &sh) {
  const float *F = a.in + k.off;
  const uint32_t n32 = (uint32_t)k.n;
  const int nt = (int)((k.n + kInsWindow - 1) / kInsWindow);
  InsTile t = ins_tile(a, k, 0, nullptr);
  for (int c = 0; c < nt && t.k_lo < t.k_hi; ++c) {
    if (t.span > kInsTile) {  // excluded by the bin-width limit; never expected
      if (threadIdx.x == 0) atomicOr(a.status, LYAF_STATUS_DOMAIN);
      return;
    }
    const uint32_t base = t.base;
    const auto src = [&](int x) -> double { return (double)tile_flux(F, n32, base, x); };
    double acc[kInsPerLane];
    const double Z = convolve_tile(a, k, t.span, src, acc, sh);
    finish_tile(a, k, t, acc, Z, sh.s, sh.red);
    const InsTile tn = ins_tile(a, k, c + 1, &t);
    t = tn;
  }
}

// The part of a skewer that a wave takes: slot i is part i mod parts of item
// i / parts.
struct InsSlot {
  int s, part;  // skewer (none: -1)
};
__device__ __forceinline__ InsSlot ins_slot(const int2 *items, int64_t n_items, int parts) {
  const int64_t i = (int64_t)blockIdx.x * kInsWaves +
                    __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  InsSlot t = {-1, 0};
  if (i < n_items * parts) {
    const uint32_t item = (uint32_t)i / (uint32_t)parts;  // i < 2^31
    t.s = __builtin_amdgcn_readfirstlane(items[item].x);
    t.part = (int)((uint32_t)i - item * (uint32_t)parts);
  }
  return t;
}

// Workgroup b, of as many as there are skewers: its waves take slots 4b .. 4b + 3
// while those last, and then, together, skewer b if its taps do not fit a wave.  (Its
// own 2 or 4 skewers in turn instead, with fewer workgroups, left a last round of
// workgroups half empty: 10000 skewers of 1000 pixels and 1.2 tap blocks, forward and
// backward, 531 us against 491.)
__global__ __launch_bounds__(kInsThreads)
__attribute__((amdgpu_waves_per_eu(4))) void instrument_kernel(
    InsArgs a, const int2 *__restrict__ items, int64_t n_items, int parts) {
  __shared__ InsLds lds;
  const InsSlot t = ins_slot(items, n_items, parts);
  const int wv = threadIdx.x >> 6;
  const int own = __builtin_amdgcn_readfirstlane(items[blockIdx.x].x);
  const auto one_block = [](const InsSkewer &k) { return 2 * k.M + 1 <= kInsTapBlock; };
  const InsSkewer ko = ins_skewer(a, own);
  if (t.s >= 0) {
    const InsSkewer k = ins_skewer(a, t.s);
    if (!k.ok && (threadIdx.x & 63) == 0) atomicOr(a.status, LYAF_STATUS_DOMAIN);
    if (k.ok && one_block(k))
      ins_forward_pieces(a, k, lds.p.w[wv], lds.p.h[wv], t.part, parts);
  }
  if (!ko.ok || one_block(ko)) return;
  __syncthreads();  // every wave is done with the LDS
  ins_forward_wide(a, ko, lds.w);
}

// Adjoint of the binning for the cnt (<= 8) consecutive pixels i0 .. i0 + cnt
// - 1 of one image range: the gradient reaching each from the bins over it,
// overlap times the bin's gradient over the bin width, summed over the
// pixel's images that meet [x_first, x_last).  A merge walk: the current bin,
// its edges and its gradient carry from pixel to pixel, so each is formed
// once per run.  out(p, h) receives pixel i0 + p.
struct InsBinGeom {
  double x_first, x_last;  // lower edges of bin 0 and of bin n_out, pixels
  double nd, inv_nd;       // n and 1 / n
};
template <class GLoad, class Out>
__device__ inline void bin_adjoint_run(const InsArgs &a, const InsSkewer &k, const InsBinGeom &G,
                                       int64_t i0, int cnt, GLoad gload, Out out) {
  double acc[8];
#pragma unroll
  for (int p = 0; p < 8; ++p) acc[p] = 0.0;
  // images y = i + L n of the run's pixels that meet the bins (a quotient
  // rounded across an integer only drops or adds an image whose overlap is
  // below 1e-9 px, or zero)
  const double L_lo = ceil((G.x_first - (double)(i0 + cnt - 1) - 1.0) * G.inv_nd);
  const double L_hi = floor((G.x_last - (double)i0) * G.inv_nd);
  for (double L = L_lo; L <= L_hi; L += 1.0) {
    const double y0 = (double)i0 + L * G.nd;
    int64_t kb = (int64_t)floor((y0 - G.x_first) * k.inv_q) - 1;
    if (kb < 0) kb = 0;
    if (kb >= k.n_out) continue;
    double e0 = bin_edge(a, k, kb), e1 = bin_edge(a, k, kb + 1);
    while (e1 <= y0 && kb + 1 < k.n_out) {  // to the first bin that ends past y0
      ++kb;
      e0 = e1;
      e1 = bin_edge(a, k, kb + 1);
    }
    double gk = (double)gload(kb) * k.inv_q;
#pragma unroll
    for (int p = 0; p < 8; ++p) {
      if (p < cnt) {
        const double y = y0 + (double)p;
        while (kb < k.n_out && e0 < y + 1.0) {
          const double ov = fmin(y + 1.0, e1) - fmax(y, e0);
          if (ov > 0.0) acc[p] = __builtin_fma(ov, gk, acc[p]);
          if (e1 > y + 1.0) break;  // the bin continues into the next pixel
          if (++kb < k.n_out) {
            e0 = e1;
            e1 = bin_edge(a, k, kb + 1);
            gk = (double)gload(kb) * k.inv_q;
          }
        }
      }
    }
  }
#pragma unroll
  for (int p = 0; p < 8; ++p)
    if (p < cnt) out(p, acc[p]);
}

// LDS of the per-tile backward when the taps fit one block: the binning
// adjoint of the tile's staged pixels (FP32, planes as in the forward) and the
// taps.  That kernel takes the skewers with more than kInsBwdBins bins (read
// from memory) or none; the per-skewer kernel below takes the others.
constexpr int kInsBwdBins = 4096;
struct InsBwdShared {
  float f[8 * kTileRows];
  double h[kInsTapBlock];
  double red[kInsThreads / 64];
};

union InsBwdLds {
  InsShared w;     // wide line-spread functions
  InsBwdShared d;  // taps in one block
};

// Backward: the adjoint of the binning at the tile's staged pixels, then the
// same line-spread convolution (the taps are even, so the adjoint convolves
// with them too).  Taps in one block: each thread forms the binning adjoint of
// eight consecutive staged pixels (one row of the eight planes) by the merge
// walk; wider line-spread functions form it pixel by pixel, block by block.
__global__ __launch_bounds__(kInsThreads) void instrument_backward_kernel(
    InsArgs a, const int2 *__restrict__ items) {
  __shared__ InsBwdLds lds;
  const int2 item = items[blockIdx.x];
  const InsSkewer k = ins_skewer(a, item.x);
  if (!k.ok) {
    if (item.y == 0 && threadIdx.x == 0) atomicOr(a.status, LYAF_STATUS_DOMAIN);
    return;
  }
  const int64_t p0 = (int64_t)item.y * kInsTile;
  const int span = (int)min<int64_t>(kInsTile, k.n - p0);
  float *gF = a.out + k.off;
  if (k.n_out == 0) {
    for (int t = threadIdx.x; t < span; t += kInsThreads) gF[p0 + t] = 0.0f;
    return;
  }
  InsBinGeom G;
  G.nd = (double)(int)k.n;
  G.inv_nd = 1.0 / G.nd;
  G.x_first = bin_edge(a, k, 0);
  G.x_last = bin_edge(a, k, k.n_out);
  const float *g = a.in + k.out_off;
  const auto g_global = [&](int64_t kb) -> float { return g[kb]; };
  const uint32_t n32 = (uint32_t)k.n;
  const uint32_t base = (uint32_t)wrap_index(p0 - k.M, (int)k.n);
  const int T = 2 * k.M + 1;
  double acc[kInsPerLane];
  double Z;
  if (T <= kInsTapBlock) {
    InsBwdShared &d = lds.d;
    const int tbp = (T + 15) & ~15;
    const double z_part = stage_taps(a, k, 0, T, tbp, d.h);
    const int rows = (span + tbp - 1 + 7) >> 3;  // staged offsets read by outputs < span
    for (int r = threadIdx.x; r < rows; r += kInsThreads) {
      // staged offsets 8r .. 8r + 7 are pixels (base + x) mod n, consecutive
      // up to the end of the box
      uint32_t i = base + 8u * (uint32_t)r;
      if (i >= n32) i -= n32;
      if (i >= n32) i %= n32;
      int done = 0;
      while (done < 8) {
        const int c = min(8 - done, (int)(n32 - i));
        const int x0 = 8 * r + done;
        bin_adjoint_run(a, k, G, (int64_t)i, c, g_global, [&](int p, double v) {
          const int x = x0 + p;
          d.f[(x & 7) * kTileRows + (x >> 3)] = (float)v;
        });
        done += c;
        i = 0;
      }
    }
    Z = block_sum_d(z_part, d.red);  // its barriers publish the staged values and the taps
#pragma unroll
    for (int q = 0; q < kInsPerLane; ++q) acc[q] = 0.0;
    if ((int)(threadIdx.x & ~63u) * kInsPerLane < span)
      conv_walk<kTileRows>(tbp, acc, d.f + threadIdx.x, d.h);
  } else {
    const auto src = [&](int x) -> double {
      uint32_t i = base + (uint32_t)x;
      if (i >= n32) i -= n32;
      if (i >= n32) i %= n32;
      double v = 0.0;
      bin_adjoint_run(a, k, G, (int64_t)i, 1, g_global, [&](int, double h) { v = h; });
      return v;
    };
    Z = convolve_tile(a, k, span, src, acc, lds.w);
  }
  const double invZ = 1.0 / Z;
  const int t0 = threadIdx.x * kInsPerLane;
#pragma unroll
  for (int q = 0; q < kInsPerLane; ++q)
    if (t0 + q < span) gF[p0 + t0 + q] = (float)(acc[q] * invZ);
}

// Backward, one workgroup per skewer whose bins fit LDS (the per-tile kernel
// takes the skewers with more bins or none).  The binning adjoint of pixel
// [y, y + 1) (pixel coordinates, one image of the pixel) is C(y + 1) - C(y),
// where C is the integral of the bins' gradient density g_k / (bin width) from
// the first bin's lower edge, in pixel units: C = P[k] + t (P[k+1] - P[k]) at
// bin coordinate k + t (t in [0, 1); a pixel is 1 / q bin units, so the
// difference carries the 1 / q), with the prefix sums P[k] = sum_{k' < k} g_k'
// (C is 0 before the first bin and P[n_out] past the last), summed over the
// pixel's images that meet the bins.  P (FP64, n_out + 1 values, dynamic LDS)
// and the taps' sum are formed once; the skewer's tiles of kInsTile pixels are
// walked, each thread forming the adjoint of rows of eight staged pixels (tile
// + taps, FP32 in planes as in the per-tile kernel) and the tile convolved
// block of taps by block.  A wave whose staged window is all zero (pixels that
// no bin reaches within the taps) stores zeros without convolving.
struct InsBwdSkShared {
  float f[8 * kTileRows];
  double h[kInsTapBlock];
  double red[kInsThreads / 64];
  double tot[kInsThreads / 64];
  uint8_t nz_row[kTileRows];  // row r of the staged block holds a nonzero value
};
constexpr int kBwdPerThread = kInsBwdBins / kInsThreads;  // bins per thread in the prefix sums
static_assert(kBwdPerThread * kInsThreads == kInsBwdBins, "the prefix sums cover every bin");
constexpr int kBwdLaneBins = 10;  // bins per lane of a wave's piece at most
constexpr int kBwdPieceDoubles = 640;  // a wave's share of P at least
static_assert(8 * kPieceRows * sizeof(float) <= kBwdPieceDoubles * sizeof(double),
              "a staged piece must fit");
static_assert(64 + kInsTapBlock / 8 <= 128, "a wave's staged rows are two per lane at most");
static_assert((kInsTile + kInsTapBlock) / 8 <= kInsThreads + kInsThreads / 8,
              "the staged rows past one per thread are at most one pixel per thread");

// The backward of one wave, taps in one block: pieces part, part + parts, .. of
// kInsPiece pixels.  The binning adjoint at the piece's staged pixels needs the prefix sums of
// the bins over them alone (differences of C do not see the sum's start): per image
// of the box that meets the bins, the lanes sum runs of consecutive bins, the wave
// scans the runs, and a lane takes C at the nine edges of its row of eight staged
// pixels and at both edges of the few staged pixels past the 64 rows.  lds holds cap
// doubles: the prefix sums, then the staged values.
__device__ __forceinline__ void ins_backward_pieces(const InsArgs &a, const InsSkewer &k,
                                                    double *lds, double *taps, int part,
                                                    int parts) {
  constexpr int kPast = kInsTapBlock / 64;
  const int lane = threadIdx.x & 63;
  const int T = 2 * k.M + 1, tbp = (T + 7) & ~7;
  const int n = (int)k.n, nt = (n + kInsPiece - 1) / kInsPiece;
  const double nd = (double)n, inv_nd = wave_uniform(1.0 / nd);
  const double x_first = wave_uniform(bin_edge(a, k, 0));
  const double x_last = wave_uniform(bin_edge(a, k, k.n_out));
  const int nb = (int)k.n_out;
  const float *g = a.in + k.out_off;
  float *st = reinterpret_cast<float *>(lds);
  const bool aligned = (((uintptr_t)(a.out + k.off)) & 15u) == 0;
  // The bins of one image of the box over a piece's staged pixels.
  struct Image {
    double L, L_hi;  // this image and the last one that meets the bins
    double t0;       // bin coordinate of the first staged pixel's lower edge
    int k0, cnt;     // bins over the staged pixels
  };
  const auto image = [&](int c, double L, double L_hi) {
    Image im;
    const int need = min(kInsPiece, n - c * kInsPiece) + tbp - 1;
    im.L = L;
    im.L_hi = L_hi;
    im.t0 = wave_uniform((__builtin_fma(L, nd, (double)(c * kInsPiece - k.M)) - x_first) *
                         k.inv_q);
    const double t1 = __builtin_fma((double)need, k.inv_q, im.t0);
    im.k0 = __builtin_amdgcn_readfirstlane((int)fmin(fmax(floor(im.t0), 0.0), (double)nb));
    im.cnt =
        __builtin_amdgcn_readfirstlane((int)fmin(fmax(floor(t1) + 1.0, 0.0), (double)nb)) - im.k0;
    return im;
  };
  const auto first_image = [&](int c) {
    // images y = s0 + x + L n of the staged pixels that meet the bins
    const int need = min(kInsPiece, n - c * kInsPiece) + tbp - 1;
    const double s0 = (double)(c * kInsPiece - k.M);
    return image(c, wave_uniform(ceil((x_first - (s0 + (double)need)) * inv_nd)),
                 wave_uniform(floor((x_last - s0) * inv_nd)));
  };
  float v[kBwdLaneBins];
  const auto load = [&](const Image &im) {
    const int m = (im.cnt + 63) >> 6;  // bins per lane, <= kBwdLaneBins (none: im.cnt <= 0)
#pragma unroll
    for (int r = 0; r < kBwdLaneBins; ++r) {
      v[r] = 0.0f;
      if (r < m) v[r] = g[im.k0 + min(m * lane + r, im.cnt - 1)];
    }
  };
  if (part >= nt) return;
  Image im = first_image(part);
  load(im);
  const double invZ = wave_taps(a, k, taps);  // while the first piece's bins are on their way
  for (int c = part; c < nt; c += parts) {
    const int p0 = c * kInsPiece, span = min(kInsPiece, n - p0);
    const int need = span + tbp - 1;
    double G[8], Gx[kPast];
#pragma unroll
    for (int p = 0; p < 8; ++p) G[p] = 0.0;
#pragma unroll
    for (int p = 0; p < kPast; ++p) Gx[p] = 0.0;
    for (;;) {
      if (im.cnt > 0 && im.L <= im.L_hi) {
        const int m = (im.cnt + 63) >> 6;
  #pragma unroll
        for (int r = 0; r < kBwdLaneBins; ++r)
          if (r < m && m * lane + r >= im.cnt) v[r] = 0.0f;
        double run = 0.0;
  #pragma unroll
        for (int r = 0; r < kBwdLaneBins; ++r)
          if (r < m) run += (double)v[r];
        double s = wave_below_d(wave_scan_d(run));
        wave_lds_order();
        double *P = lds + m * lane;
        P[0] = s;
  #pragma unroll
        for (int r = 0; r < kBwdLaneBins; ++r)
          if (r < m) {
            s += (double)v[r];
            if (r + 1 < m || lane == 63) P[r + 1] = s;
          }
        wave_lds_order();
        const int cnt = im.cnt;
        const double tc = wave_uniform(im.t0 - (double)im.k0), top = wave_uniform((double)cnt);
        int ln = lane;
        asm volatile("" : "+v"(ln));  // the pixels' FP64 edges are not kept across pieces
        const auto cum = [&](int x) -> double {  // C at the lower edge of staged pixel x
          const double t = fmin(fmax(__builtin_fma((double)x, k.inv_q, tc), 0.0), top);
          const int kb = min((int)t, cnt - 1);
          const double *q = lds + kb;
          return __builtin_fma(t - (double)kb, q[1] - q[0], q[0]);
        };
        double c0 = cum(8 * ln);
  #pragma unroll
        for (int p = 0; p < 8; ++p) {
          const double c1 = cum(8 * ln + p + 1);
          G[p] += c1 - c0;
          c0 = c1;
          if (p == 2 || p == 5) __builtin_amdgcn_sched_barrier(0);  // few in flight: registers
        }
  #pragma unroll
        for (int p = 0; p < kPast; ++p)
          if (kInsPiece + 64 * p < need) {
            const int x = kInsPiece + 64 * p + ln;
            Gx[p] += cum(x + 1) - cum(x);
          }
      }
      if (im.L >= im.L_hi) break;
      im = image(c, wave_uniform(im.L + 1.0), im.L_hi);
      load(im);
    }
    bool any = false;
    wave_lds_order();
#pragma unroll
    for (int p = 0; p < 8; ++p) {
      const float v = (float)G[p];
      any |= v != 0.0f;
      st[p * kPieceRows + lane] = v;
    }
#pragma unroll
    for (int p = 0; p < kPast; ++p)
      if (kInsPiece + 64 * p < need) {
        const float v = (float)Gx[p];
        any |= v != 0.0f;
        st[(lane & 7) * kPieceRows + ((kInsPiece + 64 * p + lane) >> 3)] = v;
      }
    wave_lds_order();
    double acc[kInsPerLane];
#pragma unroll
    for (int q = 0; q < kInsPerLane; ++q) acc[q] = 0.0;
    if (__any(any)) conv_walk<kPieceRows>(tbp, acc, st + lane, taps);
    if (c + parts < nt) {  // the next piece's bins
      im = first_image(c + parts);
      load(im);
    }
    float *o = a.out + k.off + p0 + kInsPerLane * lane;
    float f[kInsPerLane];
#pragma unroll
    for (int q = 0; q < kInsPerLane; ++q) f[q] = (float)(acc[q] * invZ);
    if (aligned && kInsPerLane * lane + 7 < span) {
      *reinterpret_cast<float4 *>(o) = make_float4(f[0], f[1], f[2], f[3]);
      *reinterpret_cast<float4 *>(o + 4) = make_float4(f[4], f[5], f[6], f[7]);
    } else {
#pragma unroll
      for (int q = 0; q < kInsPerLane; ++q)
        if (kInsPerLane * lane + q < span) o[q] = f[q];
    }
  }
}

// The backward of a skewer by the workgroup together.
__device__ void ins_backward_skewer(const InsArgs &a, const InsSkewer &k, InsBwdSkShared &sh,
                                    double *P) {
  const int nb = (int)k.n_out;
  const float *g = a.in + k.out_off;
  // P[j + 1] = sum_{j' <= j} g_j': thread t sums bins 16t .. 16t + 15, then the
  // workgroup scans the threads' totals
  double v[kBwdPerThread];
  const int j0 = (int)threadIdx.x * kBwdPerThread;
#pragma unroll
  for (int j = 0; j < kBwdPerThread; ++j) v[j] = j0 + j < nb ? (double)g[j0 + j] : 0.0;
  const int T = 2 * k.M + 1;
  const bool one_block = T <= kInsTapBlock;
  // the taps' sum (and, when they fit one block, the taps themselves)
  double z_part = 0.0;
  if (one_block) {
    z_part = stage_taps(a, k, 0, T, (T + 15) & ~15, sh.h);
  } else {
    const double scale = tap_scale(a, k);
    for (int u = threadIdx.x; u < T; u += kInsThreads) z_part += tap_value(a, k, k.M - u, scale);
  }
#pragma unroll
  for (int j = 1; j < kBwdPerThread; ++j) v[j] += v[j - 1];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  double incl = v[kBwdPerThread - 1];
  for (int d = 1; d < 64; d <<= 1) {
    const double o = __shfl_up(incl, d);
    if (lane >= d) incl += o;
  }
  if (lane == 63) sh.tot[wv] = incl;
  double excl = __shfl_up(incl, 1);
  if (lane == 0) excl = 0.0;
  __syncthreads();
  for (int w = 0; w < wv; ++w) excl += sh.tot[w];
  if (threadIdx.x == 0) P[0] = 0.0;
#pragma unroll
  for (int j = 0; j < kBwdPerThread; ++j)
    if (j0 + j < nb) P[j0 + j + 1] = excl + v[j];
  const double invZ = 1.0 / block_sum_d(z_part, sh.red);  // its barriers publish P and the taps

  const double x_first = bin_edge(a, k, 0), x_last = bin_edge(a, k, k.n_out);
  const double nd = (double)(int)k.n, inv_nd = 1.0 / nd;
  const double Ptot = P[nb];
  const auto cum = [&](double y) -> double {
    const double t = (y - x_first) * k.inv_q;
    if (!(t > 0.0)) return 0.0;
    if (t >= (double)nb) return Ptot;
    const int kb = (int)t;
    return __builtin_fma(t - (double)kb, P[kb + 1] - P[kb], P[kb]);
  };
  const uint32_t n32 = (uint32_t)k.n;
  float *gF = a.out + k.off;
  const int n_tiles = (int)((k.n + kInsTile - 1) / kInsTile);
  bool first = true;  // no barrier owed to earlier readers of f and h
  for (int c = 0; c < n_tiles; ++c) {
    const int64_t p0 = (int64_t)c * kInsTile;
    const int span = (int)min<int64_t>(kInsTile, k.n - p0);
    const bool wave_active = (int)(threadIdx.x & ~63u) * kInsPerLane < span;
    double acc[kInsPerLane];
#pragma unroll
    for (int q = 0; q < kInsPerLane; ++q) acc[q] = 0.0;
    for (int u0 = 0; u0 < T; u0 += kInsTapBlock) {
      const int tb = min(kInsTapBlock, T - u0);  // real taps in this block
      const int tbp = (tb + 15) & ~15;           // walked taps (zero-padded)
      if (!first) __syncthreads();  // every wave is done with the previous block's values
      first = false;
      if (!one_block) stage_taps(a, k, u0, tb, tbp, sh.h);
      // staged offset x is pixel (p0 - M + u0 + x) mod n
      const uint32_t base = (uint32_t)wrap_index(p0 - k.M + u0, (int)k.n);
      const int rows = (span + tbp - 1 + 7) >> 3;  // staged offsets read by outputs < span
      // the gathered gradients of cnt consecutive pixels from pixel i (no wrap
      // inside the run), at staged offsets x0 .. x0 + cnt - 1; true if any is
      // nonzero
      const auto gather = [&](const uint32_t i, const int cnt, const int x0) -> bool {
        double G[8];
#pragma unroll
        for (int p = 0; p < 8; ++p) G[p] = 0.0;
        // images y = i + L n of the run's pixels that meet [x_first, x_last)
        const double L_lo = ceil((x_first - (double)(i + cnt - 1) - 1.0) * inv_nd);
        const double L_hi = floor((x_last - (double)i) * inv_nd);
        for (double L = L_lo; L <= L_hi; L += 1.0) {
          const double y0 = __builtin_fma(L, nd, (double)i);
          double c0 = cum(y0);
#pragma unroll
          for (int p = 0; p < 8; ++p) {
            if (p < cnt) {
              const double c1 = cum(y0 + (double)(p + 1));
              G[p] += c1 - c0;
              c0 = c1;
            }
          }
        }
        bool any = false;
#pragma unroll
        for (int p = 0; p < 8; ++p) {
          if (p < cnt) {
            const int x = x0 + p;
            const float gv = (float)G[p];
            any |= gv != 0.0f;
            sh.f[(x & 7) * kTileRows + (x >> 3)] = gv;
          }
        }
        return any;
      };
      const auto wrap_px = [&](uint32_t i) {
        if (i >= n32) i -= n32;
        if (i >= n32) i %= n32;
        return i;
      };
      // staged offsets 8r .. 8r + 7 (pixels consecutive up to the end of the
      // box) for the first kInsThreads rows, one row per thread; the rows past
      // those (rows <= kInsThreads + kInsTapBlock / 8) one pixel per thread, so
      // that no thread gathers two rows while the others wait at the barrier
      if ((int)threadIdx.x < rows) {
        const int r = threadIdx.x;
        uint32_t i = wrap_px(base + 8u * (uint32_t)r);
        int done = 0;
        bool any = false;
        while (done < 8) {  // a box shorter than the row wraps more than once
          const int cnt = min(8 - done, (int)(n32 - i));
          any |= gather(i, cnt, 8 * r + done);
          done += cnt;
          i = 0;
        }
        sh.nz_row[r] = any ? 1 : 0;
      }
      if (rows > kInsThreads) {
        const int x = 8 * kInsThreads + (int)threadIdx.x;  // one pixel
        const bool in = x < 8 * rows;
        const bool nz = in && gather(wrap_px(base + (uint32_t)x), 1, x);
        // a row's 8 pixels sit on 8 consecutive lanes of one wave
        const uint64_t bal = __ballot(nz);
        if (in && (lane & 7) == 0) sh.nz_row[x >> 3] = ((bal >> (lane & ~7)) & 0xFFu) ? 1 : 0;
      }
      __syncthreads();
      // rows 64 w .. 64 w + 63 + tbp / 8 feed wave w's outputs
      const int r0 = (int)(threadIdx.x & ~63u) + lane;
      const int r1 = r0 + 64;
      const bool mine = (r0 < rows && sh.nz_row[r0]) ||
                        (lane <= tbp / 8 - 1 && r1 < rows && sh.nz_row[r1]);
      if (wave_active && __any(mine)) conv_walk<kTileRows>(tbp, acc, sh.f + threadIdx.x, sh.h);
    }
    const int t0 = threadIdx.x * kInsPerLane;
#pragma unroll
    for (int q = 0; q < kInsPerLane; ++q)
      if (t0 + q < span) gF[p0 + t0 + q] = (float)(acc[q] * invZ);
  }
}

// Four waves per SIMD (at most 128 VGPRs), as many as the LDS of a skewer
// with up to ~2700 bins leaves room for.  Dynamic LDS: the prefix sums of a skewer, or
// the waves' pieces.
__global__ __launch_bounds__(kInsThreads) __attribute__((amdgpu_waves_per_eu(4))) void
instrument_backward_skewer_kernel(InsArgs a, const int2 *__restrict__ items, int64_t n_items,
                                  int parts, int lds_doubles) {
  __shared__ InsBwdSkShared sh;
  extern __shared__ double P[];
  static_assert(sizeof(sh.f) >= kInsWaves * kInsTapBlock * sizeof(double), "the waves' taps");
  const InsSlot t = ins_slot(items, n_items, parts);
  const int wv = threadIdx.x >> 6;
  const int cap = lds_doubles / kInsWaves;
  // taps in one block and the bins over a staged piece within the wave's share of P
  const auto by_wave = [&](const InsSkewer &k) {
    const int T = 2 * k.M + 1, tbp = (T + 7) & ~7;
    const double most = fmin((double)k.n_out, (double)(kInsPiece + tbp) * k.inv_q + 3.0);
    return T <= kInsTapBlock && most <= (double)min(64 * kBwdLaneBins, cap - 65);
  };
  const int own = __builtin_amdgcn_readfirstlane(items[blockIdx.x].x);
  const InsSkewer ko = ins_skewer(a, own);
  if (t.s >= 0) {
    const InsSkewer k = ins_skewer(a, t.s);
    if (!k.ok && (threadIdx.x & 63) == 0) atomicOr(a.status, LYAF_STATUS_DOMAIN);
    if (k.ok && by_wave(k))
      ins_backward_pieces(a, k, P + wv * cap,
                          reinterpret_cast<double *>(sh.f) + wv * kInsTapBlock, t.part, parts);
  }
  if (!ko.ok || by_wave(ko)) return;
  __syncthreads();  // every wave is done with the LDS
  ins_backward_skewer(a, ko, sh, P);
}

// Parts of a skewer, a wave each, 1, 2 or 4 so that a workgroup holds whole skewers:
// four up to 2047 skewers, which otherwise leave waves' places empty, fewer beyond, as
// each part reads the skewer's constants and forms its taps.  4096 skewers of 4096 at
// 2 km/s, forward and backward: one part 68.9 and 65.0, two 70.1 and 64.4, four 76.5
// and 69.3 us (of 2047 50.3 and 44.2, 38.6 and 36.2, 41.7 and 38.0); two up to 8191,
// so that the last round of waves is never a whole skewer each.  One for boxes of a few
// hundred pixels at most, whose skewers have one piece (2000 of 200).
int ins_parts(int64_t n_items, int64_t max_n) {
  if (n_items >= 8192 || (n_items >= 1024 && max_n < kInsTapBlock)) return 1;
  return n_items >= 2048 ? 2 : 4;
}

// Workgroups: one per skewer, which may take the workgroup, or as many as the waves'
// slots fill where none can (by_waves: boxes whose taps and bins always fit a wave).
// The idle workgroups cost 20000 skewers of 300 pixels 12 of 62 us forward.
unsigned ins_grid(int64_t n_items, int parts, bool by_waves) {
  return (unsigned)(by_waves ? (n_items * parts + kInsWaves - 1) / kInsWaves : n_items);
}

}  // namespace

bool ins_bwd_skewer_item(int64_t n, int64_t n_out) {
  return n > 0 && n_out > 0 && n_out <= kInsBwdBins;
}

int ins_items_per_skewer(int64_t n, int64_t n_out, bool backward) {
  if (n <= 0) return 0;
  if (backward)  // skewers with 1 .. kInsBwdBins bins go to the per-skewer kernel
    return ins_bwd_skewer_item(n, n_out) ? 0 : (int)((n + kInsTile - 1) / kInsTile);
  return n_out > 0 ? 1 : 0;  // the forward takes a whole skewer per workgroup
}

hipError_t launch_instrument(const InsArgs &a, const int2 *items, int64_t n_items,
                             const int2 *skewer_items, int64_t n_skewer_items, int max_bins,
                             int64_t max_n, bool backward, hipStream_t st) {
  if (backward) {
    // each skewer is taken by exactly one of the two kernels
    if (n_skewer_items > 0) {
      const int lds = std::max(max_bins + 1, kInsWaves * kBwdPieceDoubles);
      const int parts = ins_parts(n_skewer_items, max_n);
      const bool by_waves = max_n < kInsTapBlock && max_bins + 65 <= kBwdPieceDoubles;
      hipLaunchKernelGGL(instrument_backward_skewer_kernel,
                         dim3(ins_grid(n_skewer_items, parts, by_waves)), dim3(kInsThreads),
                         sizeof(double) * (size_t)lds, st, a, skewer_items, n_skewer_items, parts,
                         lds);
    }
    if (n_items > 0)
      hipLaunchKernelGGL(instrument_backward_kernel, dim3((unsigned)n_items), dim3(kInsThreads),
                         0, st, a, items);
  } else if (n_items > 0) {
    const int parts = ins_parts(n_items, max_n);
    hipLaunchKernelGGL(instrument_kernel,
                       dim3(ins_grid(n_items, parts, max_n < kInsTapBlock)), dim3(kInsThreads), 0,
                       st, a, items, n_items, parts);
  }
  return hipGetLastError();
}

}  // namespace lyaf
