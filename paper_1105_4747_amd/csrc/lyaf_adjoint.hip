// lyaf_adjoint.hip -- hand-written adjoint of the optical-depth sum (Greig,
// Bolton & Wyithe 2011, Section 2.3, eqs. 4-6), by the chain rule.
//
// For source j (weight w_j, Doppler parameter b_j, t = d_ij sqrt(log2 e) / b_j,
// so that exp(-x^2) = exp2(-t^2) with x = d_ij / b_j):
//   S0_j = w_j sum_i g_i E_ij,  S1_j = w_j sum_i g_i E_ij x_ij,
//   S2_j = w_j sum_i g_i E_ij x_ij^2,  Q_j = S2_j - 1.2 S0_j,
//   dL/dv_j = 2 S1_j / b_j,
//   dL/dDelta_j = [2 S0_j + (gamma-1) [Delta_j <= pivot] Q_j] / Delta_j,
//   dL/dT0 = sum_j Q_j / T0,   dL/dgamma = sum_j Q_j ln D_j.
// The 1.2 is the temperature exponent of w (n_HI ~ T^-0.7 over b ~ T^0.5).
//
// One workgroup per 512 sources; the target gradients g_i within reach are staged
// in LDS.  Each lane owns one source at a time and walks its own run of targets,
// which starts at the target nearest its line centre less H, H uniform over the
// wave (the lanes' largest half window): target less centre is the same integer
// m on every lane, t = m a + t_c with a = dv r and |t_c| <= a / 2, and the run is
// no longer than the widest of 64 neighbouring lines.  Per block of eight targets
// the Gaussian follows a product recurrence outwards from two of them (four exp2), and
// the sums are moments about the block's middle, B_n = sum_k k^n g E, folded every 16
// targets into FP64 moments in m, from which
//   sum g E t = a M1 + t_c M0,  sum g E t^2 = a^2 M2 + 2 a t_c M1 + t_c^2 M0
// (M1 is signed and cancels across the line centre).  A wave with a line too
// narrow for the recurrence evaluates every exp2, over its window in steps of four
// targets (4096 skewers of 1024 pixels, a backward pass, with blocks of eight about the
// centre and so: 73 and 67 us at 9 km/s, 65 and 59 at 18, 91 and 84 at 5; 61, 52 and
// 76 with eight waves per SIMD and the present reach pass).  Short or wide skewers sum
// over every target with the minimal image chosen per pair.  The per-skewer T0/gamma
// terms are summed in FP64 per workgroup and then per skewer in a fixed order.  Bound by VALU issue: 4096 skewers of 2048 pixels at 2 km/s, forward and
// backward, 474 us (546 with an exp2 per pair); 20 less with a recurrence outwards from the
// middle alone (three exp2), which is not kept for its errors.  Errors against 64 bits over 16 seeds at twelve settings of 1 to 18 km/s, relative
// to the direct form's: velocity 0.80-0.95, density 0.82-0.93, gamma 0.92-1.00, T0 0.96-1.02;
// from the middle alone gamma 1.02-1.15 and T0 1.01-1.06, as its E kept the mean error
// of 4.75 exp2.
#include <math.h>

#include <type_traits>

#include "lyaf_internal.h"

namespace lyaf {

__device__ __forceinline__ float aexp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float alog2(float x) { return __builtin_amdgcn_logf(x); }

constexpr int kAdjThreads = 256;
constexpr int kAdjPasses = kTauTile / kAdjThreads;  // sources per thread of an item
constexpr int kAdjChunk = 2048;                     // targets staged in LDS at once
constexpr int kAdjMargin = 12;                      // staged targets beyond the reach
constexpr float kAdjMaxA = 0.25f;                   // coarsest grid of the recurrence
constexpr float kAdjMaxExp = 120.f;                 // exponent of the recurrence's ratio
// The hardware's exp2 is 3.2e-9 too small on average (gfx950, 2^22 arguments in each of
// nine ranges between -10 and 0.5), which every sum of the gradients' would keep; an E
// of the recurrence holds three exp2 on average.
constexpr double kAdjChainMean = 1.0 + 3.0 * 3.2e-9;

__device__ __forceinline__ int adj_wave_max(int x) {
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) x = max(x, __shfl_xor(x, m));
  return x;
}
static_assert(kTauTile % kAdjThreads == 0, "work items hold whole adjoint passes");

// 1 / x to about 1e-15 relative, x normal (the hardware's estimate and two Newton
// steps).
__device__ __forceinline__ double adj_rcp(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = fma(r, fma(-x, r, 1.0), r);
  return fma(r, fma(-x, r, 1.0), r);
}

// c 2^y to FP32's exp2 and a first-order term for the part of y that its argument drops.
__device__ __forceinline__ double adj_scaled_exp2(float c, double y) {
  const float yh = (float)y;
  const double e = (double)c * (double)aexp2(yh);
  return fma(e, kLn2 * (y - (double)yh), e);
}
// A source: r (not rounded), a = dv r rounded once, w times that rounding (a line's
// integral over the targets goes as w / a), log2 D.
struct AdjSource {
  double w, r;
  float a, l2D;
};
__device__ __forceinline__ AdjSource adj_source(const SkewerConst &K, float pivot, float delta) {
  AdjSource s = {0.0, K.R, 0.f, 0.f};
  if (delta > 0.f) {
    const float D = fmaxf(fminf(delta, pivot), 1e-30f);
    s.l2D = alog2(D);
    const double x = (double)K.gm1 * (double)s.l2D;
    s.r = adj_scaled_exp2(K.R, kTempExpR * x);
    const double a = (double)K.dv * s.r;
    s.a = (float)a;
    // w a_f / a: the rounding is below 2^-24 of a, so its ratio needs no more than FP32
    const float corr = (float)((double)s.a - a) * __builtin_amdgcn_rcpf(s.a);
    const double w = (double)delta * (double)delta * adj_scaled_exp2(K.W, kTempExpW * x);
    s.w = fma(w, (double)corr, w);
  }
  return s;
}

// Windowed sums of one source over the staged targets (gl[p] the gradient at the
// target nearest its centre): S0, S1, S2 = sum g E t^n.  Blocks of eight targets
// m = 8 i - 4 .. 8 i + 3, the line's centre in the block i = 0, whose moments are
// then taken about the centre itself: a narrow line's M1 and M2 are not
// differences of moments about a far target.
__device__ __forceinline__ void adjoint_run(const float *gl, int p, int H, float a, float tc,
                                            double &S0, double &S1, double &S2) {
  double M0 = 0.0, M1 = 0.0, M2 = 0.0;
  const int left = (H + 3) >> 3, right = (H + 4) >> 3;  // blocks beside the central one
  const float C = aexp2(-2.f * a * a), C4 = aexp2(-8.f * a * a);
  float B0, B1, B2;  // moments about the first block's middle, up to two blocks
  // the eight targets around m = 8 i, added to the moments about 8 (i - O)
  const auto block = [&](auto O, int i) {
    const float *g8 = gl + p + 8 * i - 4;
    const float fi = (float)(8 * i);
    float e[8];
    // outwards from k = 2 and k = 6, so that no ratio is raised above its square:
    // E_(k+1) = E_k U_k and E_(k-1) = E_k D_k, both falling by C per step outwards
    const float t2 = __builtin_fmaf(fi - 2.f, a, tc), t6 = __builtin_fmaf(fi + 2.f, a, tc);
    e[2] = aexp2(-(t2 * t2));
    e[6] = aexp2(-(t6 * t6));
    const float U2 = aexp2(-(__builtin_fmaf(2.f, t2, a) * a));
    const float D6 = aexp2(__builtin_fmaf(2.f, t6, -a) * a);
    const float U6 = U2 * C4, D2 = D6 * C4;
    e[3] = e[2] * U2;
    e[1] = e[2] * D2;
    e[0] = e[1] * (D2 * C);
    e[7] = e[6] * U6;
    e[5] = e[6] * D6;
    e[4] = e[5] * (D6 * C);
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const float gE = g8[k] * e[k];
      constexpr float o = 8.f * (float)decltype(O)::value - 4.f;
      const float kk = o + (float)k;
      if (decltype(O)::value == 0 && k == 0) {
        B0 = gE;
        B1 = kk * gE;
        B2 = kk * kk * gE;
      } else {
        B0 += gE;
        if (kk != 0.f) {
          B1 = __builtin_fmaf(gE, kk, B1);
          B2 = __builtin_fmaf(gE, kk * kk, B2);
        }
      }
    }
  };
  const auto fold = [&](int i) {  // moments about 8 i, to moments about the centre
    const double b0 = B0, b1 = B1, md = (double)(8 * i);
    M0 += b0;
    M1 += fma(md, b0, b1);
    M2 += fma(md, fma(md, b0, 2.0 * b1), (double)B2);
  };
  const std::integral_constant<int, 0> first;
  const std::integral_constant<int, 1> second;
  int i = -left;
  if (left & 1) {  // the central block is then the first of a pair
    block(first, i);
    fold(i);
    ++i;
  }
  for (; i < right; i += 2) {
    block(first, i);
    block(second, i + 1);
    fold(i);
  }
  if (i == right) {
    block(first, i);
    fold(i);
  }
  M0 *= kAdjChainMean;
  M1 *= kAdjChainMean;
  M2 *= kAdjChainMean;
  const double ad = a, td = tc;
  S0 = M0;
  S1 = fma(ad, M1, td * M0);
  S2 = fma(ad * ad, M2, td * fma(2.0 * ad, M1, td * M0));
}

// The same with an exp2 per pair, for waves with a line too narrow for the recurrence:
// the targets m = -H .. H, four to a step, as the whole window may be no wider than a
// block of eight (5 to 12 targets each side between 18 and 8 km/s); sums of 16 folded
// into FP64.
__device__ __forceinline__ void adjoint_pairs(const float *gl, int p, int H, float a, float tc,
                                              double &S0, double &S1, double &S2) {
  S0 = S1 = S2 = 0.0;
  const float *gp = gl + p - H;
  const int steps = (2 * H + 4) >> 2;
  for (int st = 0; st < steps; st += 4) {
    float s0 = 0.f, s1 = 0.f, s2 = 0.f;
    const int end = min(st + 4, steps);
    for (int q = st; q < end; ++q) {
      const float t0 = __builtin_fmaf((float)(4 * q - H), a, tc);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const float t = k == 0 ? t0 : __builtin_fmaf((float)k, a, t0);
        const float tt = t * t;
        const float gE = gp[4 * q + k] * aexp2(-tt);
        s0 += gE;
        s1 = __builtin_fmaf(gE, t, s1);
        s2 = __builtin_fmaf(gE, tt, s2);
      }
    }
    S0 += (double)s0;
    S1 += (double)s1;
    S2 += (double)s2;
  }
}

// The same over every target, the minimal image chosen per pair; gl is filled
// chunk by chunk.
__device__ void adjoint_full(const SkewerConst &K, const float *__restrict__ g, float *gl, int j,
                             float v, float r, double &S0, double &S1, double &S2) {
  const int n = K.n;
  const float dv = K.dv, nf = (float)n;
  const float invV = 1.f / (nf * dv);
  S0 = S1 = S2 = 0.0;
  for (int c0 = 0; c0 < n; c0 += kAdjChunk) {
    const int cn = min(kAdjChunk, n - c0);
    __syncthreads();
    for (int c = threadIdx.x; c < cn; c += kAdjThreads) gl[c] = g[c0 + c];
    __syncthreads();
    for (int c16 = 0; c16 < cn; c16 += 16) {
      float s0 = 0.f, s1 = 0.f, s2 = 0.f;
      const float fj = (float)(c0 + c16 - j);
      const auto pair = [&](int k) {
        const float fd = fj + (float)k;
        const float d0 = __builtin_fmaf(fd, dv, -v);
        const float img = floorf(__builtin_fmaf(d0, invV, 0.5f));
        const float d = __builtin_fmaf(__builtin_fmaf(img, -nf, fd), dv, -v);
        const float t = d * r;
        const float gE = gl[c16 + k] * aexp2(-(t * t));
        const float gEt = gE * t;
        s0 += gE;
        s1 += gEt;
        s2 = __builtin_fmaf(gEt, t, s2);
      };
      if (c16 + 16 <= cn) {
#pragma unroll
        for (int k = 0; k < 16; ++k) pair(k);
      } else {
#pragma unroll 1
        for (int k = 0; k < cn - c16; ++k) pair(k);
      }
      S0 += (double)s0;
      S1 += (double)s1;
      S2 += (double)s2;
    }
  }
}

// Eight waves per SIMD (64 VGPRs, none spilled): few targets a line leave a wave waiting
// on its loads (78 VGPRs, 4096 x 1024 pixels of 18 km/s: 45.9 us, 43.7 so; of 3 km/s
// 89.8 and 85.1; 4096 x 2048 of 2 km/s 201 and 196).
__global__ __launch_bounds__(kAdjThreads) __attribute__((amdgpu_waves_per_eu(8))) void
tau_adjoint_kernel(Batch b, const int2 *__restrict__ items, const float *__restrict__ g,
                   float *__restrict__ gdelta, float *__restrict__ gvpec,
                   double *__restrict__ gpart) {
  __shared__ float gl[kAdjChunk];
  __shared__ double shd[8];
  const int2 item = items[blockIdx.x];
  const SkewerConst K = b.skc[item.x];
  const int64_t off = b.offsets[item.x];
  const int n = K.n;
  const int j0 = item.y * kTauTile;
  const int j_end = min(j0 + kTauTile, n);
  float dd[kAdjPasses], vv[kAdjPasses];
  bool bad = false;
#pragma unroll
  for (int p = 0; p < kAdjPasses; ++p) {
    const int j = j0 + p * kAdjThreads + (int)threadIdx.x;
    dd[p] = j < j_end ? b.delta[off + j] : 0.f;
    vv[p] = j < j_end ? b.vpec[off + j] : 0.f;
  }
  // staged margin: a run reaches at most vpx + half from its source, and its outer
  // blocks up to 8 more.  A box of at least two half windows of 6 b or more holds
  // one image of every pair that matters (the others' terms are below exp(-36)), if
  // the velocities reach less than the box; a window of less than 6 b ends where the
  // terms matter, so such a box has to hold two reaches.
  const int RH = K.vpx + K.half + kAdjMargin;
  const bool one_image = b.window_k >= 6.f
                             ? 2 * K.half + 8 <= n && K.vpx < n
                             : 2 * ((K.reach + kAdjMargin + 3) & ~3) + 8 <= n;
  const bool windowed = kTauTile + 2 * RH <= kAdjChunk && one_image;
  if (windowed) {
    const int cnt = (j_end - j0) + 2 * RH;
    const float *gs = g + off;
    for (int c = threadIdx.x; c < cnt; c += kAdjThreads) {
      int i = j0 - RH + c;
      while (i < 0) i += n;
      while (i >= n) i -= n;
      gl[c] = gs[i];
    }
  }
  __syncthreads();
  double q_T0 = 0.0, q_gam = 0.0;
#pragma unroll 1
  for (int p = 0; p < kAdjPasses; ++p) {
    const int j = j0 + p * kAdjThreads + (int)threadIdx.x;
    if (j0 + p * kAdjThreads >= j_end) break;
    const float delta = p == 0 ? dd[0] : dd[kAdjPasses - 1], v = p == 0 ? vv[0] : vv[kAdjPasses - 1];
    static_assert(kAdjPasses <= 2, "a source each from dd and vv");
    // an invalid density sets the sticky domain bit (the reach pass may not
    // have read Delta)
    bad |= !(delta >= 0.f) || !isfinite(delta);
    const AdjSource s = adj_source(K, b.pivot, delta);
    double S0, S1, S2;
    if (windowed) {
      const bool line = s.w > 0.0;
      const float a = line ? s.a : 0.f, r = (float)s.r;
      // the target nearest the centre, and the centre's distance from it: exact to
      // one rounding of a value below dv
      const float vs = line ? fminf(fmaxf(rintf(v * K.inv_dv), (float)-K.vpx), (float)K.vpx) : 0.f;
      const float tc = line ? __builtin_fmaf(vs, K.dv, -v) * r : 0.f;
      const float h = b.window_k * (float)kSqrtLog2e * K.inv_dv / r;  // k b / dv
      const int Hl = line ? (int)fminf(h + 0.51f, (float)K.half) : 0;
      const int H = __builtin_amdgcn_readfirstlane(adj_wave_max(Hl));
      const bool wide = !(a <= kAdjMaxA) || !(2.f * a * a * ((float)H + 11.f) <= kAdjMaxExp);
      const int at = (j - j0) + RH + (int)vs;
      if (__any(wide))
        adjoint_pairs(gl, at, H, a, tc, S0, S1, S2);
      else
        adjoint_run(gl, at, min(H + 1, K.half), a, tc, S0, S1, S2);
    } else {
      adjoint_full(K, g + off, gl, j, v, (float)s.r, S0, S1, S2);
    }
    if (j < j_end) {
      float gd = 0.f, gv = 0.f;
      if (s.w > 0.0) {
        // t = x sqrt(log2 e) and 1/b = r / sqrt(log2 e); Q = S2 - 1.2 S0 cancels
        // where x^2 ~ 1.2: formed in FP64
        const double w = s.w;
        const double Q = w * (S2 * (1.0 / kLog2e) - 1.2 * S0);
        gv = (float)(2.0 * w * S1 * s.r * (1.0 / kLog2e));
        const double below = (delta <= b.pivot) ? (double)K.gm1 : 0.0;
        gd = (float)(fma(below, Q, 2.0 * w * S0) * adj_rcp((double)delta));
        q_T0 += Q;
        q_gam += Q * ((double)s.l2D * kLn2);  // Q ln D
      }
      gdelta[off + j] = gd;
      gvpec[off + j] = gv;
    }
  }
  if (__any(bad) && (threadIdx.x & 63) == 0) atomicOr(b.status, LYAF_STATUS_DOMAIN);
  // FP64 workgroup sums of Q (for dL/dT0 after division by T0) and Q ln D
  double a0 = q_T0, a1 = q_gam;
  for (int m = 32; m >= 1; m >>= 1) {
    a0 += __shfl_xor(a0, m);
    a1 += __shfl_xor(a1, m);
  }
  const int wv = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
    shd[wv] = a0;
    shd[4 + wv] = a1;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    gpart[2 * (int64_t)blockIdx.x + 0] = (shd[0] + shd[1]) + (shd[2] + shd[3]);
    gpart[2 * (int64_t)blockIdx.x + 1] = (shd[4] + shd[5]) + (shd[6] + shd[7]);
  }
}

// Per-skewer fixed-order sum of the workgroup partials.  Items of skewer s are
// item_base[s] .. item_base[s+1]-1.
__global__ void adjoint_skewer_sum_kernel(const double *__restrict__ gpart,
                                          const int64_t *__restrict__ item_base,
                                          const float *__restrict__ T0, int64_t S,
                                          double *__restrict__ gT0,
                                          double *__restrict__ ggamma) {
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= S) return;
  double q = 0.0, ql = 0.0;
  for (int64_t k = item_base[s]; k < item_base[s + 1]; ++k) {
    q += gpart[2 * k + 0];
    ql += gpart[2 * k + 1];
  }
  if (gT0) gT0[s] = q / (double)T0[s];
  if (ggamma) ggamma[s] = ql;
}

hipError_t launch_tau_adjoint(const Batch &b, const int2 *items, int64_t n_items,
                              const int64_t *item_base_dev, const float *g, float *gdelta,
                              float *gvpec, double *gT0, double *ggamma, double *gpart,
                              hipStream_t st) {
  if (n_items > 0)
    hipLaunchKernelGGL(tau_adjoint_kernel, dim3((unsigned)n_items), dim3(kAdjThreads), 0, st, b,
                       items, g, gdelta, gvpec, gpart);
  if (b.n_skewers > 0 && (gT0 || ggamma))
    hipLaunchKernelGGL(adjoint_skewer_sum_kernel, dim3((unsigned)((b.n_skewers + 255) / 256)),
                       dim3(256), 0, st, gpart, item_base_dev, b.T0, b.n_skewers, gT0, ggamma);
  return hipGetLastError();
}

}  // namespace lyaf
