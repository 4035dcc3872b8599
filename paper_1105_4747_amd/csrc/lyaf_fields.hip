// lyaf_fields.hip -- skewer-only synthesis of the linear density and velocity
// fields (Greig, Bolton & Wyithe 2011, Section 2.1 and Appendix B).
//
// A Gaussian field g(k) is given on the half-spectrum of a real N^3 grid of a
// periodic box of side L (k = 2 pi (mx, my, mz) / L, mx and my signed, mz = 0 ..
// N/2).  The dark-matter field is delta_DM = amp sqrt(P(|k|)) g, with P
// linearly interpolated from a table; the baryons follow the filter of eq. (1),
// delta_b = delta_DM / (1 + k^2 / k_F^2); the velocity follows eq. (3),
// v = E_+ i k / k^2 delta_DM, of which the component along the sight-lines (z)
// is kept.  Only the S requested sight-lines (columns (x_s, y_s)) are brought
// back to real space, as Appendix B does it: transforms across the (kx, ky)
// planes, then one 1D transform per sight-line.  For each field F:
//
//   f_s(z) = N^-3 sum_mz c_mz Re[ C_s(mz) e^{2 pi i mz z / N} ],  c = 1 at mz = 0, N/2, else 2,
//   C_s(mz) = sum_mx e^{2 pi i mx x_s / N} T(mx, y_s, mz),
//   T(mx, y, mz) = sum_my e^{2 pi i my y / N} F(mx, my, mz).
//
// Grids of 512 and 1024 with enough sight-lines go through field_planes_kernel,
// which does both transforms across (kx, ky) one mz at a time without an
// intermediate, and field_z_planes_kernel.  Otherwise three kernels, all reading
// their inputs once:
//   field_ky_kernel  persistent workgroups over (mx, run of C consecutive mz)
//                    items, the next item's modes read ahead: reads the
//                    N x C modes (C consecutive mz are contiguous), forms both
//                    fields' spectra (FP32 multipliers), inverse-transforms
//                    the 2C columns along my in LDS as one batch (FP32,
//                    Stockham passes) and
//                    writes only the rows y that some sight-line uses:
//                    T [rows][N][N/2+1] complex float per field;
//   field_kx_kernel  one workgroup per (group of up to 8 sight-lines sharing a
//                    row y, 256 consecutive mz): each thread owns one mz and
//                    sums over mx for every sight-line of the group, in FP64,
//                    twiddles from an LDS table: C [S][N/2+1] complex double;
//   field_z_kernel   one workgroup per sight-line: both real fields as the real
//                    and imaginary parts of one complex inverse transform
//                    (Hermitian extension of each half-spectrum), FP64 in LDS,
//                    scaled by N^-3 and stored as float.
#include <algorithm>

#include "lyaf_fft.h"
#include "lyaf_internal.h"

namespace lyaf {
namespace {

constexpr int kKyThreads = 1024;
constexpr int kKyCap = 16384;  // N 2C complex floats in LDS (128 KB)
constexpr int kKxThreads = 256;
constexpr int kKxLines = kFieldLinesPerGroup;  // sight-lines per group
constexpr int kZThreads = 256;

// Multiplier of g for each field at integer wavenumber (mx, my, mz): the
// baryon field's real factor and the velocity's real factor (times i).
__device__ inline void field_factors(const FieldArgs &a, int mx, int my, int mz, float &fb,
                                     float &fv) {
  const int m2 = mx * mx + my * my + mz * mz;  // exact: at most 3 (N/2)^2
  const float m2f = (float)m2;
  const float kmag = a.kfun * __builtin_sqrtf(m2f);
  const float x = kmag * a.inv_dk;
  const int j = (int)x;  // x >= 0
  float P = 0.f;
  if (j + 1 < a.n_table) {
    const float p0 = (float)a.pk[j], p1 = (float)a.pk[j + 1];
    P = __builtin_fmaf(x - (float)j, p1 - p0, p0);
  } else if (j + 1 == a.n_table && x == (float)j) {
    P = (float)a.pk[j];  // exactly at the last node
  }
  const float A = a.amp * __builtin_sqrtf(fmaxf(P, 0.f));
  fb = A / __builtin_fmaf(a.kfun2_inv_kF2, m2f, 1.f);
  fv = (m2 > 0) ? a.E_over_kfun * (float)mz / m2f * A : 0.f;
}

// Persistent: workgroup b takes items b', b' + G, .. (G workgroups; b' puts
// the workgroups of one XCD on consecutive items, whose mz runs share cache
// lines), and reads the next item's modes into registers while the current
// one is transformed and stored.
__global__ __launch_bounds__(kKyThreads) void field_ky_kernel(FieldArgs a, int lgC,
                                                               int n_chunks) {
  // [N][2][C]: both fields' C columns side by side, one batch of 2C transforms
  extern __shared__ float2 lds_ky[];
  const int N = a.N, H = a.H;
  const int C = 1 << lgC;
  const int n_items = N * n_chunks;
  const int n_el = N << lgC;
  const int G = (int)gridDim.x;  // a multiple of 8
  const int first = ((int)blockIdx.x & 7) * (G >> 3) + ((int)blockIdx.x >> 3);
  constexpr int E = kKyCap / 2 / kKyThreads;  // modes per thread per item
  float2 nxt[E];
  auto fetch = [&](int item) {
    const int kx = item / n_chunks;
    const int kz0 = (item - kx * n_chunks) * C;
    const float2 *src = a.modes + (size_t)kx * N * H + kz0;
    int tx = (int)threadIdx.x;
    asm volatile("" : "+v"(tx));
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int q = tx + e * kKyThreads;
      nxt[e] = make_float2(0.f, 0.f);
      if (q < n_el && kz0 + (q & (C - 1)) < H) nxt[e] = src[(size_t)(q >> lgC) * H + (q & (C - 1))];
    }
  };
  if (first < n_items) fetch(first);
  for (int item = first; item < n_items; item += G) {
    const int kx = item / n_chunks;
    const int kz0 = (item - kx * n_chunks) * C;
    const int mx = kx <= N / 2 ? kx : kx - N;
    // the per-element indices below are recomputed for every item: hoisted out
    // of the item loop they would hold E sets of registers for its whole length
    int tx = (int)threadIdx.x;
    asm volatile("" : "+v"(tx));
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int q = tx + e * kKyThreads;
      if (q < n_el) {
        const int ky = q >> lgC, c = q & (C - 1);
        float2 b = make_float2(0.f, 0.f), v = make_float2(0.f, 0.f);
        if (kz0 + c < H) {
          const float2 g = nxt[e];
          float fb, fv;
          field_factors(a, mx, ky <= N / 2 ? ky : ky - N, kz0 + c, fb, fv);
          // conjugated on the way in: the inverse transform is conj(FFT(conj))
          b = make_float2(g.x * fb, -g.y * fb);
          v = make_float2(-g.y * fv, -g.x * fv);  // conj(i fv g)
        }
        lds_ky[(ky << (lgC + 1)) + c] = b;
        lds_ky[(ky << (lgC + 1)) + C + c] = v;
      }
      asm volatile("" ::: "memory");  // one element's multipliers at a time
    }
    lds_barrier();
    if (item + G < n_items) fetch(item + G);  // in flight during the transform
    fft_batch<kKyThreads, kKyCap>(lds_ky, a.twiddle, N, lgC + 1);
    const int n_out = a.n_rows << (lgC + 1);
    for (int q = threadIdx.x; q < n_out; q += kKyThreads) {
      const int yi = q >> (lgC + 1), f = (q >> lgC) & 1, c = q & (C - 1);
      if (kz0 + c < H) {
        float2 *dst = (f == 0 ? a.Tb : a.Tv) + ((size_t)yi * N + kx) * H + kz0 + c;
        *dst = conj(lds_ky[(a.rows[yi] << (lgC + 1)) + (f << lgC) + c]);
      }
    }
    lds_barrier();  // every read of the buffer is done before the next item
  }
}

// e^{+2 pi i t / N} for t < N from the half-period table of e^{-2 pi i u / 4096}.
__device__ inline double2 root_of_unity(const double2 *__restrict__ T, int t, int N) {
  const int u = t * (kFftTableLen / N);
  const double2 w = (u < kFftTableLen / 2) ? T[u] : make_double2(-T[u - kFftTableLen / 2].x,
                                                                  -T[u - kFftTableLen / 2].y);
  return conj(w);
}

__global__ __launch_bounds__(kKxThreads) void field_kx_kernel(FieldArgs a, int n_kzb) {
  extern __shared__ double2 tw[];  // [N]
  const int g = (int)blockIdx.x / n_kzb;
  const int kzb = (int)blockIdx.x - g * n_kzb;
  const int N = a.N, H = a.H;
  const int4 grp = a.groups[g];  // (row, first line, count, -)
  for (int t = threadIdx.x; t < N; t += kKxThreads) tw[t] = root_of_unity(a.twiddle, t, N);
  int xs[kKxLines];
#pragma unroll
  for (int m = 0; m < kKxLines; ++m) xs[m] = m < grp.z ? a.lines[grp.y + m].y : 0;
  __syncthreads();
  const int kz = kzb * kKxThreads + (int)threadIdx.x;
  if (kz - (int)(threadIdx.x & 63) >= H) return;  // the wave holds no mz
  const bool valid = kz < H;
  const size_t base = (size_t)grp.x * N * H + (valid ? kz : 0);
  const float2 *rb = a.Tb + base;
  const float2 *rv = a.Tv + base;
  double2 ab[kKxLines], av[kKxLines];
#pragma unroll
  for (int m = 0; m < kKxLines; ++m) {
    ab[m] = make_double2(0.0, 0.0);
    av[m] = make_double2(0.0, 0.0);
  }
  int idx[kKxLines];  // (kx x_m) mod N
#pragma unroll
  for (int m = 0; m < kKxLines; ++m) idx[m] = 0;
  const int mask = N - 1;
  constexpr int U = 4;  // rows of T in flight per thread
  for (int kx0 = 0; kx0 < N; kx0 += U) {
    float2 tb[U], tv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool in = valid && kx0 + u < N;
      tb[u] = in ? rb[(size_t)(kx0 + u) * H] : make_float2(0.f, 0.f);
      tv[u] = in ? rv[(size_t)(kx0 + u) * H] : make_float2(0.f, 0.f);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const double bx = tb[u].x, by = tb[u].y, vx = tv[u].x, vy = tv[u].y;
#pragma unroll
      for (int m = 0; m < kKxLines; ++m) {
        if (m < grp.z) {
          const double2 w = tw[idx[m]];
          ab[m].x = __builtin_fma(bx, w.x, __builtin_fma(-by, w.y, ab[m].x));
          ab[m].y = __builtin_fma(bx, w.y, __builtin_fma(by, w.x, ab[m].y));
          av[m].x = __builtin_fma(vx, w.x, __builtin_fma(-vy, w.y, av[m].x));
          av[m].y = __builtin_fma(vx, w.y, __builtin_fma(vy, w.x, av[m].y));
          idx[m] = (idx[m] + xs[m]) & mask;
        }
      }
    }
  }
  if (!valid) return;
#pragma unroll
  for (int m = 0; m < kKxLines; ++m) {
    if (m < grp.z) {
      const size_t s = (size_t)a.lines[grp.y + m].x;
      a.Cb[s * H + kz] = ab[m];
      a.Cv[s * H + kz] = av[m];
    }
  }
}

// The planes of one mz at a time, straight from the modes to the sight-lines'
// sums over mx: T is neither written nor read.  A workgroup keeps FP64 sums of
// both fields for up to kFieldSlots sight-lines per thread in registers, and
// takes four pairs mx = p, -p per round (p = 0 stands for the pair 0, N/2): each
// wave reads one mx column of modes (the next round's while the sight-lines are
// summed), forms both fields' spectra, and transforms them along my by itself
// (wave_fft, no workgroup barriers); then every thread adds the eight columns to
// its sight-lines,
//   C += cos (T(p) + T(-p)) + i sin (T(p) - T(-p)),
// four FP64 FMAs per pair and field for both signs of mx, with the sums and
// differences formed once per row.  Sight-lines of a row are consecutive slots
// of a thread.  The modes of one mz lie 8 bytes in each row of the grid, so the
// workgroups of an XCD hold consecutive mz and run in step: a line of the
// modes serves 16 of them from one L2.  At n = 1024 and 6250 sight-lines the
// kernel takes 6.3 ms, the my and mx kernels through T 6.7 + 5.3; without its
// reads of modes it takes 3.9 (contiguous reads of the same bytes: 4.1), so the
// gather bounds it.  Measured and not kept: reads of two mz at once with the odd
// one's modes kept in memory for its own turn (6.2 ms for 2 GB), the reads
// started before the transforms (6.5), the waves' reads in rotated order (6.3).
// Workgroup g of G takes planes mz = g, g + G, .. below N/2; the last plane
// N/2, which would leave most of a round idle, is split over the workgroups by
// mx, its parts added by field_last_kernel in a fixed order.
template <int E>
struct FieldPlanesLds {
  static constexpr int N = 64 * E;
  float2 col[8][2][N];   // by wave: mx = +-(4 r + wave / 2); both fields
  double2 tw[N];         // e^{-2 pi i t / N}
  float2 tw1[kWaveTw1<E>], tw2[kWaveTw2];
};

template <int E, int K>
__global__ __launch_bounds__(kFieldThreads) __attribute__((amdgpu_waves_per_eu(2))) void
field_planes_kernel(FieldArgs a) {
  constexpr int N = 64 * E, HALF = N / 2;
  constexpr int ROUNDS = HALF / 4;
  extern __shared__ double2 lds_planes[];
  FieldPlanesLds<E> &sh = *reinterpret_cast<FieldPlanesLds<E> *>(lds_planes);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  for (int t = tid; t < N; t += kFieldThreads) sh.tw[t] = conj(root_of_unity(a.twiddle, t, N));
  wave_fft_tables<E>(sh.tw1, sh.tw2, a.twiddle, tid, kFieldThreads);

  // this thread's slots: x | last-of-row flag << 11 | LDS position of y << 12
  uint32_t word[K];
  double br[K], bi[K], vr[K], vi[K];  // conjugates of the sums, both fields
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const uint32_t w = a.slot_words[k * kFieldThreads + tid];
    word[k] = (w & 0xFFFu) | ((uint32_t)wave_fft_pos<E>((int)(w >> 12)) << 12);
    br[k] = bi[k] = vr[k] = vi[k] = 0.0;
  }

  const int G = (int)gridDim.x;
  const int g = (G & 7) == 0 ? ((int)blockIdx.x & 7) * (G >> 3) + ((int)blockIdx.x >> 3)
                             : (int)blockIdx.x;
  const int n_planes = g < HALF ? (HALF - g + G - 1) / G : 0;
  const int n_last = g < ROUNDS ? (ROUNDS - g + G - 1) / G : 0;
  const int n_steps = n_planes * ROUNDS + n_last;
  // step i: (mz, round)
  const auto step_of = [&](int i, int &mz, int &r) {
    const int pl = i / ROUNDS;
    mz = pl < n_planes ? g + pl * G : HALF;
    r = pl < n_planes ? i - pl * ROUNDS : g + (i - n_planes * ROUNDS) * G;
  };
  const int pair = wave >> 1;
  const bool minus = (wave & 1) != 0;
  float2 gm[E];  // modes of this wave's column, elements lane + 64 r
  const auto fetch = [&](int i) {
    int mz, r;
    step_of(i, mz, r);
    const int p = 4 * r + pair;
    const int kx = p == 0 ? (minus ? HALF : 0) : (minus ? N - p : p);
    int ln = lane;
    asm volatile("" : "+v"(ln));  // addresses per step, not held across the steps
    const float2 *src = a.modes + ((size_t)kx * N + ln) * a.H + mz;
#pragma unroll
    for (int e = 0; e < E; ++e) gm[e] = src[(size_t)(64 * e) * a.H];
  };
  float2 *colb = sh.col[wave][0], *colv = sh.col[wave][1];
  if (n_steps > 0) fetch(0);
  __syncthreads();  // the tables
  for (int i = 0; i < n_steps; ++i) {
    int mz, r;
    step_of(i, mz, r);
    {
      const int p = 4 * r + pair;
      const int mx = p == 0 ? (minus ? HALF : 0) : p;  // |mx|: the factors hold its square
      // factors of |my| = 0 .. N/2, each formed once per column: element y uses
      // |my| = y below N/2 and N - y above, which another lane holds
      float2 *fac = colb;
      int ln = lane;
      asm volatile("" : "+v"(ln));  // addresses per step, not held across the steps
#pragma unroll
      for (int j = 0; j <= E / 2; ++j) {
        const int my = j < E / 2 ? ln + 64 * j : HALF;
        float fb, fv;
        field_factors(a, mx, my, mz, fb, fv);
        if (j < E / 2 || ln == 0) fac[my] = make_float2(fb, fv);
        asm volatile("" ::: "memory");  // one factor at a time
      }
      asm volatile("" ::: "memory");
      float2 x[E];
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const int y = ln + 64 * e;
        const float2 f = fac[e < E / 2 ? y : N - y];
        // conjugated on the way in: the inverse transform is conj(FFT(conj))
        x[e] = make_float2(gm[e].x * f.x, -gm[e].y * f.x);
        colv[y] = make_float2(-gm[e].y * f.y, -gm[e].x * f.y);  // conj(i fv g), kept in LDS
        if ((e & 3) == 3) asm volatile("" ::: "memory");
      }
      wave_fft<E>(x, colb, sh.tw1, sh.tw2, ln);
      asm volatile("" ::: "memory");
#pragma unroll
      for (int e = 0; e < E; ++e) x[e] = colv[ln + 64 * e];
      asm volatile("" ::: "memory");
      wave_fft<E>(x, colv, sh.tw1, sh.tw2, ln);
    }
    lds_barrier();
    if (i + 1 < n_steps) fetch(i + 1);  // in flight during the sums
#pragma unroll 1
    for (int q = 0; q < 4; ++q) {
      const int p = 4 * r + q;
      // p = 0, columns 0 and N/2: T(0) + (-1)^x T(N/2).  The same sums give it
      // with (cos, sin) = (1, 0) or (0, 1) by the parity of x, from the table's
      // entries 0 and 3 N/4, and the row's differences turned by a quarter
      const int pm = p == 0 ? 3 * N / 4 : p;
      const uint32_t xm = p == 0 ? 1u : 0x7FFu;
      const float2 *cq = sh.col[2 * q][0];
      double bux, buy, bdx, bdy, vux, vuy, vdx, vdy;  // T(p) +- T(-p) of a row, conjugated
      const auto row = [&](uint32_t w) {
        asm volatile("" : "+v"(w));  // decoded here, not held decoded across the steps
        const float2 *c = cq + (w >> 12);
        const float2 bp = c[0], vp = c[N], bm = c[2 * N], vm = c[3 * N];
        bux = (double)bp.x + (double)bm.x;
        bdx = (double)bp.x - (double)bm.x;
        buy = (double)bp.y + (double)bm.y;
        bdy = (double)bp.y - (double)bm.y;
        vux = (double)vp.x + (double)vm.x;
        vdx = (double)vp.x - (double)vm.x;
        vuy = (double)vp.y + (double)vm.y;
        vdy = (double)vp.y - (double)vm.y;
        if (p == 0) {
          double t = bdx;
          bdx = bdy;
          bdy = -t;
          t = vdx;
          vdx = vdy;
          vdy = -t;
        }
      };
      const auto root = [&](uint32_t w) {
        asm volatile("" : "+v"(w));
        return sh.tw[(pm * (int)(w & xm)) & (N - 1)];
      };
      row(word[0]);
      double2 e = root(word[0]);
#pragma unroll
      for (int k = 0; k < K; ++k) {
        const double2 e1 = k + 1 < K ? root(word[k + 1 < K ? k + 1 : k]) : e;
        br[k] = __builtin_fma(e.x, bux, __builtin_fma(-e.y, bdy, br[k]));
        bi[k] = __builtin_fma(e.x, buy, __builtin_fma(e.y, bdx, bi[k]));
        vr[k] = __builtin_fma(e.x, vux, __builtin_fma(-e.y, vdy, vr[k]));
        vi[k] = __builtin_fma(e.x, vuy, __builtin_fma(e.y, vdx, vi[k]));
        if (k + 1 < K) {
          // the sums above are done with this row before the next one replaces it
          asm volatile("" : "+v"(br[k]), "+v"(bi[k]), "+v"(vr[k]), "+v"(vi[k]));
          if (word[k] & 0x800u) row(word[k + 1 < K ? k + 1 : k]);
        }
        e = e1;
      }
    }
    const bool end = i + 1 == n_steps || (mz < HALF && r == ROUNDS - 1);
    if (end) {
      double2 *out = mz < HALF ? a.planes + (size_t)mz * 2 * kFieldSlotSum
                               : a.last_parts + (size_t)g * 2 * kFieldSlotSum;
      int t = tid;
      asm volatile("" : "+v"(t));
#pragma unroll
      for (int k = 0; k < K; ++k) {
        out[k * kFieldThreads + t] = make_double2(br[k], -bi[k]);
        out[kFieldSlotSum + k * kFieldThreads + t] = make_double2(vr[k], -vi[k]);
        br[k] = bi[k] = vr[k] = vi[k] = 0.0;
      }
    }
    lds_barrier();  // the next round overwrites the columns
  }
}

// The last plane mz = N/2: the workgroups' parts added in order.
__global__ __launch_bounds__(256) void field_last_kernel(FieldArgs a, int parts) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= 2 * kFieldSlotSum) return;
  double2 s = make_double2(0.0, 0.0);
#pragma unroll 16
  for (int p = 0; p < parts; ++p) s = cadd(s, a.last_parts[(size_t)p * 2 * kFieldSlotSum + i]);
  a.planes[(size_t)(a.N / 2) * 2 * kFieldSlotSum + i] = s;
}

// The transform along z from the plane sums, four neighbouring slots per
// workgroup (64 contiguous bytes of every plane), as field_z_kernel.
constexpr int kZPThreads = 512;
__global__ __launch_bounds__(kZPThreads) void field_z_planes_kernel(FieldArgs a) {
  extern __shared__ double2 lds_zp[];  // [N][4]
  const int N = a.N, half = N / 2;
  const int c = threadIdx.x & 3;
  const int slot = 4 * (int)blockIdx.x + c;
  const int line = a.slot_lines[slot];
  if (!__syncthreads_or(line >= 0)) return;
  for (int k = threadIdx.x >> 2; k <= half; k += kZPThreads / 4) {
    const double2 *pl = a.planes + (size_t)k * 2 * kFieldSlotSum + slot;
    double2 b = make_double2(0.0, 0.0), v = b;
    if (line >= 0) {
      b = pl[0];
      v = pl[kFieldSlotSum];
    }
    // conjugates of C_b + i C_v and, at N - k, of conj(C_b) + i conj(C_v); the
    // imaginary parts of planes 0 and N/2 drop out of Re[]
    if (k == 0 || k == half) {
      lds_zp[4 * k + c] = make_double2(b.x, -v.x);
    } else {
      lds_zp[4 * k + c] = make_double2(b.x - v.y, -(b.y + v.x));
      lds_zp[4 * (N - k) + c] = make_double2(b.x + v.y, b.y - v.x);
    }
  }
  __syncthreads();
  fft_batch<kZPThreads, 4096>(lds_zp, a.twiddle, N, 2);
  if (line < 0) return;
  const double scale = a.inv_n3;
  float *ob = a.delta_b + (size_t)line * N;
  float *ov = a.v_z + (size_t)line * N;
  for (int t = threadIdx.x >> 2; t < N; t += kZPThreads / 4) {
    const double2 z = lds_zp[4 * t + c];  // conj of the inverse transform: f_b - i f_v
    ob[t] = (float)(z.x * scale);
    ov[t] = (float)(-z.y * scale);
  }
}

__global__ __launch_bounds__(kZThreads) void field_z_kernel(FieldArgs a) {
  extern __shared__ double2 lds_z[];  // [N]
  const int s = blockIdx.x;
  const int N = a.N, H = a.H, half = N / 2;
  const double2 *cb = a.Cb + (size_t)s * H;
  const double2 *cv = a.Cv + (size_t)s * H;
  for (int k = threadIdx.x; k < N; k += kZThreads) {
    double2 z;
    if (k == 0 || k == half) {
      z = make_double2(cb[k].x, cv[k].x);  // the imaginary parts drop out of Re[]
    } else if (k < half) {
      const double2 b = cb[k], v = cv[k];
      z = make_double2(b.x - v.y, b.y + v.x);  // C_b + i C_v
    } else {
      const double2 b = cb[N - k], v = cv[N - k];
      z = make_double2(b.x + v.y, v.x - b.y);  // conj(C_b) + i conj(C_v)
    }
    lds_z[k] = conj(z);
  }
  __syncthreads();
  fft_batch<kZThreads, kFieldMaxN>(lds_z, a.twiddle, N, 0);
  const double scale = a.inv_n3;
  float *ob = a.delta_b + (size_t)s * N;
  float *ov = a.v_z + (size_t)s * N;
  for (int t = threadIdx.x; t < N; t += kZThreads) {
    const double2 z = lds_z[t];  // conj of the inverse transform: f_b - i f_v
    ob[t] = (float)(z.x * scale);
    ov[t] = (float)(-z.y * scale);
  }
}

bool g_attr_set[64] = {false};

}  // namespace

int field_ky_columns(int N) { return std::min(16, kKyCap / (2 * N)); }

int g_ky_resident[64] = {0};

hipError_t field_kernel_attributes(int *ky_resident) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
  if (g_attr_set[dev]) {
    *ky_resident = g_ky_resident[dev];
    return hipSuccess;
  }
  if ((e = hipFuncSetAttribute((const void *)field_ky_kernel,
                               hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)(sizeof(float2) * kKyCap))) != hipSuccess)
    return e;
  if ((e = hipFuncSetAttribute((const void *)field_z_kernel,
                               hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)(sizeof(double2) * kFieldMaxN))) != hipSuccess)
    return e;
  int per_cu = 0, cus = 0;
  if ((e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void *)field_ky_kernel,
                                                        kKyThreads,
                                                        sizeof(float2) * kKyCap)) != hipSuccess ||
      (e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev)) !=
          hipSuccess)
    return e;
  g_ky_resident[dev] = std::max(1, per_cu) * cus;
  g_attr_set[dev] = true;
  *ky_resident = g_ky_resident[dev];
  return hipSuccess;
}

bool field_planes_fit(int N, int64_t n_lines) {
  // 512 and 1024 are the sizes of wave_fft; the slots hold 6656 sight-lines.  A
  // call at N = 512 takes 0.83, 0.89, 0.99 and 1.27 ms with 16, 400, 1500 and
  // 6250 sight-lines against 0.92, 1.26, 1.55 and 2.46 through T; at N = 1024
  // the gathered modes set the time, 5.97, 5.99 and 6.90 ms with 16, 256 and
  // 6250, and T costs little while few rows are kept: 5.28, 5.92 and 12.37.
  if (n_lines > kFieldSlotSum) return false;
  return N == 512 || (N == 1024 && n_lines >= 320);
}

int field_last_parts(int N, int resident) { return std::min(N / 8, resident); }

hipError_t field_planes_attributes(int N, int *resident) {
  static int known[64][2] = {{0}};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
  int &r = known[dev][N == 1024 ? 1 : 0];
  if (r == 0) {
    const void *f = N == 1024 ? (const void *)field_planes_kernel<16, kFieldSlots>
                              : (const void *)field_planes_kernel<8, kFieldSlots>;
    const size_t lds = N == 1024 ? sizeof(FieldPlanesLds<16>) : sizeof(FieldPlanesLds<8>);
    int per_cu = 0, cus = 0;
    if ((e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds)) !=
            hipSuccess ||
        (e = hipFuncSetAttribute((const void *)field_z_planes_kernel,
                                 hipFuncAttributeMaxDynamicSharedMemorySize,
                                 (int)(4 * 1024 * sizeof(double2)))) != hipSuccess ||
        (e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, f, kFieldThreads, lds)) !=
            hipSuccess ||
        (e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev)) !=
            hipSuccess)
      return e;
    r = std::max(1, per_cu) * cus;
  }
  *resident = r;
  return hipSuccess;
}

hipError_t launch_field_planes(const FieldArgs &a, int resident, hipStream_t st) {
  if (a.N == 1024)
    hipLaunchKernelGGL((field_planes_kernel<16, kFieldSlots>), dim3(resident), dim3(kFieldThreads),
                       sizeof(FieldPlanesLds<16>), st, a);
  else
    hipLaunchKernelGGL((field_planes_kernel<8, kFieldSlots>), dim3(resident), dim3(kFieldThreads),
                       sizeof(FieldPlanesLds<8>), st, a);
  return hipGetLastError();
}

hipError_t launch_field_last(const FieldArgs &a, int resident, hipStream_t st) {
  hipLaunchKernelGGL(field_last_kernel, dim3((2 * kFieldSlotSum + 255) / 256), dim3(256), 0, st,
                     a, field_last_parts(a.N, resident));
  return hipGetLastError();
}

hipError_t launch_field_z_planes(const FieldArgs &a, hipStream_t st) {
  hipLaunchKernelGGL(field_z_planes_kernel, dim3(kFieldSlotSum / 4), dim3(kZPThreads),
                     4 * sizeof(double2) * (size_t)a.N, st, a);
  return hipGetLastError();
}

hipError_t launch_field_ky(const FieldArgs &a, int resident, hipStream_t st) {
  const int C = field_ky_columns(a.N);
  int lgC = 0;
  while ((1 << lgC) < C) ++lgC;
  const int n_chunks = (a.H + C - 1) / C;
  const int items = a.N * n_chunks;
  // persistent: the resident workgroups, at most the items, a multiple of 8
  const int grid = std::max(8, std::min(resident, (items + 7) / 8 * 8) / 8 * 8);
  hipLaunchKernelGGL(field_ky_kernel, dim3(grid), dim3(kKyThreads),
                     sizeof(float2) * (size_t)(a.N << (lgC + 1)), st, a, lgC, n_chunks);
  return hipGetLastError();
}

hipError_t launch_field_kx(const FieldArgs &a, int n_groups, hipStream_t st) {
  const int n_kzb = (a.H + kKxThreads - 1) / kKxThreads;
  if (n_groups <= 0) return hipSuccess;
  hipLaunchKernelGGL(field_kx_kernel, dim3(n_groups * n_kzb), dim3(kKxThreads),
                     sizeof(double2) * (size_t)a.N, st, a,
                     n_kzb);
  return hipGetLastError();
}

hipError_t launch_field_z(const FieldArgs &a, int n_lines, hipStream_t st) {
  if (n_lines <= 0) return hipSuccess;
  hipLaunchKernelGGL(field_z_kernel, dim3(n_lines), dim3(kZThreads),
                     sizeof(double2) * (size_t)a.N, st, a);
  return hipGetLastError();
}

}  // namespace lyaf
