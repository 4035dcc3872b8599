// lyaf_fft.h -- in-LDS complex FFT passes shared by the kernels that transform
// along one axis (the 1D flux power spectrum, the skewer-only field synthesis,
// the 3D flux power spectrum).  Device code only; nothing here is public ABI.
//
// A batch of C transforms of N points (N, C powers of two) sits in LDS with
// element j of transform c at buf[j C + c], so that C consecutive columns of a
// global array load and store without bank conflicts.  Each Stockham pass of
// radix R reads, for butterfly (j, c) with k = j mod Ns, the R inputs
// x_r = buf[(j + r N/R) C + c], twiddles x_r by w^r, w = e^{-2 pi i k/(R Ns)},
// and after a barrier writes their length-R DFT to buf[((j - k) R + k + r Ns) C + c];
// passes of radix 8 run while 8 Ns <= N, then one of radix 4 or 2 as log2 N
// needs.  Every thread holds its butterflies' outputs in registers across the
// barrier, so the passes work in place.  The transforms are forward
// (e^{-2 pi i}); an inverse transform is the conjugate of the forward
// transform of the conjugate, which the callers apply on the way in and out.
//
// Twiddles come from one half-period table of the largest transform,
// T[t] = e^{-2 pi i t / kFftTableLen} for t < kFftTableLen / 2, held in FP64 in
// device memory (it stays in L1/L2); a transform of N points takes every
// (kFftTableLen / N)-th entry.  FP32 batches round the entry once.
#pragma once

#include <hip/hip_runtime.h>

namespace lyaf {

constexpr int kFftTableLen = 4096;  // longest transform the table serves

__device__ inline double2 cmul(double2 a, double2 b) {
  return make_double2(__builtin_fma(a.x, b.x, -a.y * b.y), __builtin_fma(a.x, b.y, a.y * b.x));
}
__device__ inline float2 cmul(float2 a, float2 b) {
  return make_float2(__builtin_fmaf(a.x, b.x, -a.y * b.y), __builtin_fmaf(a.x, b.y, a.y * b.x));
}
__device__ inline double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ inline float2 cadd(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ inline double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
__device__ inline float2 csub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
// multiply by -i and by +i
__device__ inline double2 mul_mi(double2 a) { return make_double2(a.y, -a.x); }
__device__ inline float2 mul_mi(float2 a) { return make_float2(a.y, -a.x); }
__device__ inline double2 mul_pi(double2 a) { return make_double2(-a.y, a.x); }
__device__ inline float2 mul_pi(float2 a) { return make_float2(-a.y, a.x); }
__device__ inline double2 conj(double2 a) { return make_double2(a.x, -a.y); }
__device__ inline float2 conj(float2 a) { return make_float2(a.x, -a.y); }

// Workgroup barrier for LDS traffic only: waits for this wave's LDS
// operations (lgkmcnt(0); vmcnt and expcnt left at their maxima, encoding
// 0xC07F on gfx9-family parts), then s_barrier.  Unlike __syncthreads() it
// does not wait for global loads, so reads of the next tile issued before it
// stay in flight across the transform's passes.  The empty asm statements keep
// the compiler from moving memory accesses across it.
__device__ inline void lds_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0xC07F);
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

template <typename V>
__device__ inline V twiddle_as(double2 w);
template <>
__device__ inline double2 twiddle_as<double2>(double2 w) { return w; }
template <>
__device__ inline float2 twiddle_as<float2>(double2 w) {
  return make_float2((float)w.x, (float)w.y);
}

template <typename V>
__device__ inline void dft4(V a0, V a1, V a2, V a3, V &y0, V &y1, V &y2, V &y3) {
  const V s02 = cadd(a0, a2), d02 = csub(a0, a2);
  const V s13 = cadd(a1, a3), d13 = csub(a1, a3);
  y0 = cadd(s02, s13);
  y1 = cadd(d02, mul_mi(d13));
  y2 = csub(s02, s13);
  y3 = cadd(d02, mul_pi(d13));
}

// Position of element e of a single transform of N points in LDS: the index within
// eight XORed with the number of the eight, so that the first passes' writes, eight
// elements apart, meet all of the banks (half of the LDS cycles of a 2048-point FP64
// transform were conflicts).  Steps of 64 elements leave the XOR as it is.
__device__ inline int fft_swizzle(int e, int N) { return N >= 512 ? e ^ ((e >> 3) & 7) : e; }

// One in-place pass of radix R over C = 2^lgC transforms of N points (see the
// header).  CAP bounds N C over every call of the instantiation, so each of
// the THREADS threads holds at most CAP / (R THREADS) butterflies.  A length-8
// DFT is two length-4 DFTs of x_k + x_{k+4} and (x_k - x_{k+4}) e^{-2 pi i k/8}.
// FIRST: the pass of Ns = 1 without its twiddles, which are 1.  SWZ: see fft_batch.
template <int R, int THREADS, int CAP, bool SWZ, bool FIRST, typename V>
__device__ void fft_pass(V *buf, const double2 *__restrict__ T, int N, int lgC, int Ns) {
  using S = decltype(V{}.x);
  constexpr int B = (CAP / R + THREADS - 1) / THREADS;
  const int nb = (N / R) << lgC;
  const int cmask = (1 << lgC) - 1;
  const int step = kFftTableLen / (R * Ns);  // stride in the table
  V y[B][R];
#pragma unroll
  for (int b = 0; b < B; ++b) {
    const int q = (int)threadIdx.x + b * THREADS;
    if (q < nb) {
      const int c = q & cmask;
      const int j = q >> lgC;
      const int k = j & (Ns - 1);
      V w;
      if constexpr (!FIRST) w = twiddle_as<V>(T[k * step]);
      V x[R];
#pragma unroll
      for (int r = 0; r < R; ++r)  // N / R is a multiple of 64 wherever elements are swizzled
        x[r] = buf[SWZ ? fft_swizzle(j, N) + r * (N / R) : ((j + r * (N / R)) << lgC) + c];
      if constexpr (R == 8) {
        if constexpr (!FIRST) {
          const V w2 = cmul(w, w), w3 = cmul(w2, w), w4 = cmul(w2, w2);
          const V w5 = cmul(w4, w), w6 = cmul(w3, w3), w7 = cmul(w6, w);
          x[1] = cmul(x[1], w);
          x[2] = cmul(x[2], w2);
          x[3] = cmul(x[3], w3);
          x[4] = cmul(x[4], w4);
          x[5] = cmul(x[5], w5);
          x[6] = cmul(x[6], w6);
          x[7] = cmul(x[7], w7);
        }
        constexpr S h = (S)0.70710678118654752440;  // sqrt(1/2)
        const V b0 = csub(x[0], x[4]);
        const V t1 = csub(x[1], x[5]);
        V b1;  // * (1 - i)/sqrt2
        b1.x = h * (t1.x + t1.y);
        b1.y = h * (t1.y - t1.x);
        const V b2 = mul_mi(csub(x[2], x[6]));
        const V t3 = csub(x[3], x[7]);
        V b3;  // * -(1 + i)/sqrt2
        b3.x = h * (t3.y - t3.x);
        b3.y = -h * (t3.x + t3.y);
        dft4(cadd(x[0], x[4]), cadd(x[1], x[5]), cadd(x[2], x[6]), cadd(x[3], x[7]), y[b][0],
             y[b][2], y[b][4], y[b][6]);
        dft4(b0, b1, b2, b3, y[b][1], y[b][3], y[b][5], y[b][7]);
      } else if constexpr (R == 4) {
        if constexpr (!FIRST) {
          const V w2 = cmul(w, w), w3 = cmul(w2, w);
          x[1] = cmul(x[1], w);
          x[2] = cmul(x[2], w2);
          x[3] = cmul(x[3], w3);
        }
        dft4(x[0], x[1], x[2], x[3], y[b][0], y[b][1], y[b][2], y[b][3]);
      } else {
        if constexpr (!FIRST) x[1] = cmul(x[1], w);
        y[b][0] = cadd(x[0], x[1]);
        y[b][1] = csub(x[0], x[1]);
      }
    }
    // one butterfly's inputs live at a time: without this the compiler reads
    // every butterfly's inputs first and runs out of registers at large B
    asm volatile("" ::: "memory");
  }
  lds_barrier();  // every read of this pass is done
#pragma unroll
  for (int b = 0; b < B; ++b) {
    const int q = (int)threadIdx.x + b * THREADS;
    if (q < nb) {
      const int c = q & cmask;
      const int j = q >> lgC;
      const int k = j & (Ns - 1);
      const int base = (j - k) * R + k;
      if constexpr (SWZ) {  // fft_swizzle(base + r Ns), by the forms it takes
        const bool on = N >= 512;
        const int b0 = fft_swizzle(base, N);
        if (on && FIRST) {
#pragma unroll
          for (int r = 0; r < R; ++r) buf[b0 ^ r] = y[b][r];  // R = 8
        } else if (on && Ns == 8) {
#pragma unroll
          for (int r = 0; r < R; ++r) buf[(b0 ^ r) + 8 * r] = y[b][r];
        } else {
#pragma unroll
          for (int r = 0; r < R; ++r) buf[b0 + r * Ns] = y[b][r];
        }
      } else {
#pragma unroll
        for (int r = 0; r < R; ++r) buf[((base + r * Ns) << lgC) + c] = y[b][r];
      }
    }
  }
  lds_barrier();
}

// ---------------------------------------------------------------------------
// One transform of N = 64 E points (E = 8 or 16) per wave, without workgroup
// barriers: radix E in each lane's registers, then the 64-point transforms as
// two radix-8 steps, with two exchanges through the wave's own N elements of LDS
// (a batch in passes of radix 8, 8, 8, 2 at N = 1024 exchanges four times, each
// between two barriers).  Lane l holds x[r] = element l + 64 r on entry.  The
// result, element k = k1 + E (k2 + 8 k3), is left in LDS at wave_fft_pos(k); the
// XOR of the indices keeps every access to distinct banks.  Twiddles come from
// LDS, one rounding of the FP64 table each: tw1[(k1 - 1) 64 + l] = e^{-2 pi i l
// k1/N}, tw2[(k2 - 1) 8 + a] = e^{-2 pi i a k2/64}.
__device__ inline int wave_fft_at(int k1, int b, int a) {
  return (k1 << 6) + ((b ^ (k1 & 7)) << 3) + (a ^ b);
}
template <int E>
__device__ inline int wave_fft_pos(int k) {
  return wave_fft_at(k & (E - 1), (k / E) & 7, (k / E) >> 3);
}
template <int E>
constexpr int kWaveTw1 = (E - 1) * 64;
constexpr int kWaveTw2 = 7 * 8;

// The entries t of both tables for a thread of the workgroup that fills them.
template <int E, typename V>
__device__ inline void wave_fft_tables(V *tw1, V *tw2, const double2 *__restrict__ T, int tid,
                                       int threads) {
  const auto root = [&](int t, int n) {  // e^{-2 pi i t / n}, 0 <= t < n
    const int u = t * (kFftTableLen / n);
    return twiddle_as<V>(u < kFftTableLen / 2 ? T[u]
                                              : make_double2(-T[u - kFftTableLen / 2].x,
                                                             -T[u - kFftTableLen / 2].y));
  };
  for (int i = tid; i < kWaveTw1<E>; i += threads)
    tw1[i] = root((i & 63) * ((i >> 6) + 1), 64 * E);  // below 64 (E - 1) < 64 E
  for (int i = tid; i < kWaveTw2; i += threads) tw2[i] = root((i & 7) * ((i >> 3) + 1), 64);
}

// Length-8 DFT in registers (as the radix-8 pass).
template <typename V>
__device__ inline void dft8(V (&x)[8]) {
  using S = decltype(V{}.x);
  constexpr S h = (S)0.70710678118654752440;  // sqrt(1/2)
  const V b0 = csub(x[0], x[4]);
  const V t1 = csub(x[1], x[5]);
  const V b2 = mul_mi(csub(x[2], x[6]));
  const V t3 = csub(x[3], x[7]);
  V b1, b3;
  b1.x = h * (t1.x + t1.y);
  b1.y = h * (t1.y - t1.x);
  b3.x = h * (t3.y - t3.x);
  b3.y = -h * (t3.x + t3.y);
  V y[8];
  dft4(cadd(x[0], x[4]), cadd(x[1], x[5]), cadd(x[2], x[6]), cadd(x[3], x[7]), y[0], y[2], y[4],
       y[6]);
  dft4(b0, b1, b2, b3, y[1], y[3], y[5], y[7]);
#pragma unroll
  for (int k = 0; k < 8; ++k) x[k] = y[k];
}

// Length-16 DFT in registers: length-4 DFTs over r = j, j + 4, j + 8, j + 12,
// twiddles e^{-2 pi i j k/16}, length-4 DFTs over j.
template <typename V>
__device__ inline void dft16(V (&x)[16]) {
  using S = decltype(V{}.x);
  constexpr S c1 = (S)0.92387953251128675613, s1 = (S)0.38268343236508977173;  // pi/8
  constexpr S h = (S)0.70710678118654752440;
  V t[4][4];
#pragma unroll
  for (int j = 0; j < 4; ++j)
    dft4(x[j], x[j + 4], x[j + 8], x[j + 12], t[j][0], t[j][1], t[j][2], t[j][3]);
  const auto rot = [](V a, S c, S s) {  // a (c - i s)
    V o;
    o.x = a.x * c + a.y * s;
    o.y = a.y * c - a.x * s;
    return o;
  };
  const auto rot8 = [&](V a) {  // a e^{-i pi/4}
    V o;
    o.x = h * (a.x + a.y);
    o.y = h * (a.y - a.x);
    return o;
  };
  t[1][1] = rot(t[1][1], c1, s1);
  t[1][2] = rot8(t[1][2]);
  t[1][3] = rot(t[1][3], s1, c1);
  t[2][1] = rot8(t[2][1]);
  t[2][2] = mul_mi(t[2][2]);
  t[2][3] = mul_mi(rot8(t[2][3]));
  t[3][1] = rot(t[3][1], s1, c1);
  t[3][2] = mul_mi(rot8(t[3][2]));
  t[3][3] = rot(t[3][3], -c1, -s1);
#pragma unroll
  for (int k = 0; k < 4; ++k)
    dft4(t[0][k], t[1][k], t[2][k], t[3][k], x[k], x[k + 4], x[k + 8], x[k + 12]);
}

template <int E, typename V>
__device__ inline void wave_fft(V (&x)[E], V *col, const V *tw1, const V *tw2, int lane) {
  static_assert(E == 8 || E == 16, "64 E points");
  if constexpr (E == 16)
    dft16(x);
  else
    dft8(x);
  const int lo = lane & 7, hi = lane >> 3;
  {
    const int in = lo ^ hi;  // position of a = lo within the eight of b = hi
#pragma unroll
    for (int k1 = 0; k1 < E; ++k1) {
      col[(k1 << 6) + ((hi ^ (k1 & 7)) << 3) + in] =
          k1 == 0 ? x[0] : cmul(x[k1], tw1[(k1 - 1) * 64 + lane]);
      if ((k1 & 3) == 3) asm volatile("" ::: "memory");  // four twiddles in flight
    }
  }
  // LDS accesses of one wave are performed in order: the reads below see the
  // other lanes' writes without a wait; the compiler must keep that order
  asm volatile("" ::: "memory");
#pragma unroll
  for (int u = 0; u < E / 8; ++u) {  // radix 8 over b: lane (a = lo, k1 = hi + 8u)
    V *c = col + ((hi + 8 * u) << 6);
    V y[8];
#pragma unroll
    for (int b = 0; b < 8; ++b) y[b] = c[((b ^ hi) << 3) + (lo ^ b)];
    dft8(y);
#pragma unroll
    for (int k2 = 0; k2 < 8; ++k2)
      c[((k2 ^ hi) << 3) + (lo ^ k2)] = k2 == 0 ? y[0] : cmul(y[k2], tw2[(k2 - 1) * 8 + lo]);
    asm volatile("" ::: "memory");  // one butterfly's elements at a time
  }
  asm volatile("" ::: "memory");
#pragma unroll
  for (int u = 0; u < E / 8; ++u) {  // radix 8 over a: lane (k2 = lo, k1 = hi + 8u)
    V *c = col + ((hi + 8 * u) << 6) + ((lo ^ hi) << 3);
    V y[8];
#pragma unroll
    for (int a = 0; a < 8; ++a) y[a] = c[a ^ lo];
    dft8(y);
#pragma unroll
    for (int k3 = 0; k3 < 8; ++k3) c[k3 ^ lo] = y[k3];
    asm volatile("" ::: "memory");
  }
}

// The whole forward transform of the batch (N >= 1; N = 1 is the identity).
// The caller has published buf with a barrier; the last pass ends with one
// (LDS only: global loads issued before the transform may still be in flight).
// SWZ: a single transform (lgC = 0) with element e at fft_swizzle(e, N), its first
// pass by itself (in the batches along ky that costs 60 spilled registers).
template <int THREADS, int CAP, bool SWZ = false, typename V>
__device__ void fft_batch(V *buf, const double2 *__restrict__ T, int N, int lgC) {
  int Ns = 1;
  if constexpr (SWZ) {  // the pass of Ns = 1 by itself, without its twiddles
    if (N >= 8) {
      fft_pass<8, THREADS, CAP, true, true>(buf, T, N, 0, 1);
      Ns = 8;
    } else if (N == 4) {
      fft_pass<4, THREADS, CAP, true, true>(buf, T, N, 0, 1);
      Ns = 4;
    } else if (N == 2) {
      fft_pass<2, THREADS, CAP, true, true>(buf, T, N, 0, 1);
      Ns = 2;
    }
  }
  while (Ns * 8 <= N) {
    fft_pass<8, THREADS, CAP, SWZ, false>(buf, T, N, lgC, Ns);
    Ns *= 8;
  }
  if (Ns * 4 <= N) {
    fft_pass<4, THREADS, CAP, SWZ, false>(buf, T, N, lgC, Ns);
    Ns *= 4;
  }
  if (Ns * 2 <= N) fft_pass<2, THREADS, CAP, SWZ, false>(buf, T, N, lgC, Ns);
}

}  // namespace lyaf
