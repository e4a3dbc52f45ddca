// Discrete Fourier transforms of short lines held in registers, every length and twiddle
// known at compile time (the coarsest multigrid level and the FFT solvers).
#pragma once

#include <hip/hip_runtime.h>

namespace pm_dft {

// cos and sin of 2 pi m / n at compile time, from the Taylor series about the nearest
// multiple of pi / 2 (angle at most pi / 4: 14 terms reach the last bit of a double)
constexpr double kPi = 3.14159265358979323846;
constexpr double taylor(double x, bool sine) {
  double term = sine ? x : 1.0, sum = term;
  for (int k = 1; k <= 14; ++k) {
    const int d = sine ? 2 * k * (2 * k + 1) : (2 * k - 1) * 2 * k;
    term *= -x * x / d;
    sum += term;
  }
  return sum;
}
constexpr double turn(int m, int n, bool sine) {
  m = ((m % n) + n) % n;
  const int q = (8 * m + n) / (2 * n);  // nearest quarter turn, 0 .. 4
  const double x = 2.0 * kPi * (4.0 * m - (double)q * n) / (4.0 * n);
  const double c = taylor(x, false), s = taylor(x, true);
  switch (q & 3) {
    case 0: return sine ? s : c;
    case 1: return sine ? c : -s;
    case 2: return sine ? -s : -c;
    default: return sine ? -c : s;
  }
}

// In-place DFT of N values (natural order in and out), e^{-2 pi i/N} forward, its
// conjugate inverse (INV), unnormalised: lengths that are multiples of four split into the
// four subsequences m, m + 4, .. (one layer of twiddles for two halvings: fewer roundings),
// other even ones into the even and odd elements, odd lengths summed directly.
template <int N, bool INV, bool EXACT = true>
struct Dft {
  static __device__ __forceinline__ void run(float2 (&x)[N]) {
    if constexpr (N == 2) {
      const float2 a = x[0], b = x[1];
      x[0] = make_float2(a.x + b.x, a.y + b.y);
      x[1] = make_float2(a.x - b.x, a.y - b.y);
    } else if constexpr (N % 4 == 0) {
      float2 q[4][N / 4];
#pragma unroll
      for (int m = 0; m < N / 4; ++m)
#pragma unroll
        for (int r = 0; r < 4; ++r) q[r][m] = x[4 * m + r];
      if constexpr (N > 4)
#pragma unroll
        for (int r = 0; r < 4; ++r) Dft<N / 4, INV, EXACT>::run(q[r]);
      combine4<0>(x, q);
    } else if constexpr (N % 2 == 0) {
      float2 e[N / 2], o[N / 2];
#pragma unroll
      for (int m = 0; m < N / 2; ++m) {
        e[m] = x[2 * m];
        o[m] = x[2 * m + 1];
      }
      Dft<N / 2, INV, EXACT>::run(e);
      Dft<N / 2, INV, EXACT>::run(o);
      combine<0>(x, e, o);
    } else {
      direct(x);
    }
  }
  // v e^{-+ 2 pi i K / N}. The constants carry the remainder that FP32 leaves of them: the
  // first roots of unity all round to a modulus 2.5e-8 too small, and a transform that
  // multiplies by them again and again loses amplitude by it. With radix-2 splits and rounded
  // constants the potential of a 512^3 solve was 2.37e-7 off (seven-point kernel), 256^3
  // 2.25e-7; so 1.78e-7 and 1.83e-7. Time: 256^3 solves 150 -> 151 us, dealiased
  // second-order initial conditions, bound by vector instructions, 256^3 2984 -> 3037 us.
  // Not EXACT: rounded constants, for the coarsest multigrid level, whose solution is a
  // correction and whose time is one chain of these (16^3 5.84 -> 5.45 us).
  template <int K>
  static __device__ __forceinline__ float2 turned(float2 v) {
    if constexpr (4 * K == N) {
      return INV ? make_float2(-v.y, v.x) : make_float2(v.y, -v.x);
    } else if constexpr (2 * K == N) {
      return make_float2(-v.x, -v.y);
    } else if constexpr (K > 0) {
      constexpr double cd = turn(K, N, false), sd = (INV ? 1.0 : -1.0) * turn(K, N, true);
      constexpr float c = (float)cd, s = (float)sd, cl = (float)(cd - (double)c), sl = (float)(sd - (double)s);
      if constexpr (!EXACT) {
        return make_float2(v.x * c - v.y * s, v.x * s + v.y * c);
      } else if constexpr (8 * K % N == 0) {  // +-1 +-i over the root of 2
        constexpr bool same = (cd > 0.0) == (sd > 0.0);
        const float p = same ? v.x - v.y : v.x + v.y, q = same ? v.x + v.y : v.y - v.x;
        return make_float2(fmaf(p, c, p * cl), fmaf(q, c, q * cl));
      } else {
        const float x = fmaf(-v.y, s, fmaf(v.x, cl, -(v.y * sl))), y = fmaf(v.y, c, fmaf(v.x, sl, v.y * cl));
        return make_float2(fmaf(v.x, c, x), fmaf(v.x, s, y));
      }
    } else {
      return v;
    }
  }
  template <int K>
  static __device__ __forceinline__ void combine4(float2 (&x)[N], const float2 (&q)[4][N / 4]) {
    if constexpr (K < N / 4) {
      const float2 a = q[0][K], b = turned<K>(q[1][K]), c = turned<2 * K>(q[2][K]), d = turned<3 * K>(q[3][K]);
      const float2 s = make_float2(a.x + c.x, a.y + c.y), t = make_float2(a.x - c.x, a.y - c.y);
      const float2 u = make_float2(b.x + d.x, b.y + d.y), v = make_float2(b.x - d.x, b.y - d.y);
      const float2 w = INV ? make_float2(-v.y, v.x) : make_float2(v.y, -v.x);  // (-+ i) v
      x[K] = make_float2(s.x + u.x, s.y + u.y);
      x[K + N / 4] = make_float2(t.x + w.x, t.y + w.y);
      x[K + N / 2] = make_float2(s.x - u.x, s.y - u.y);
      x[K + 3 * N / 4] = make_float2(t.x - w.x, t.y - w.y);
      combine4<K + 1>(x, q);
    }
  }
  template <int K>
  static __device__ __forceinline__ void combine(float2 (&x)[N], const float2 (&e)[N / 2],
                                                 const float2 (&o)[N / 2]) {
    if constexpr (K < N / 2) {
      float2 t = o[K];
      if constexpr (4 * K == N) {
        t = INV ? make_float2(-t.y, t.x) : make_float2(t.y, -t.x);
      } else if constexpr (K > 0) {
        constexpr float c = (float)turn(K, N, false), s = (float)(INV ? 1.0 : -1.0) * (float)turn(K, N, true);
        t = make_float2(t.x * c - t.y * s, t.x * s + t.y * c);
      }
      x[K] = make_float2(e[K].x + t.x, e[K].y + t.y);
      x[K + N / 2] = make_float2(e[K].x - t.x, e[K].y - t.y);
      combine<K + 1>(x, e, o);
    }
  }
  // odd N: the pairs x_m +- x_{N-m} halve the products
  static __device__ __forceinline__ void direct(float2 (&x)[N]) {
    float2 p[N / 2 + 1], q[N / 2 + 1], y[N];
    float2 all = x[0];
#pragma unroll
    for (int m = 1; m <= N / 2; ++m) {
      p[m] = make_float2(x[m].x + x[N - m].x, x[m].y + x[N - m].y);
      q[m] = make_float2(x[m].x - x[N - m].x, x[m].y - x[N - m].y);
      all = make_float2(all.x + p[m].x, all.y + p[m].y);
    }
    y[0] = all;
    rows<1>(x, p, q, y);
#pragma unroll
    for (int m = 0; m < N; ++m) x[m] = y[m];
  }
  template <int K>
  static __device__ __forceinline__ void rows(const float2 (&x)[N], const float2 (&p)[N / 2 + 1],
                                              const float2 (&q)[N / 2 + 1], float2 (&y)[N]) {
    if constexpr (K <= N / 2) {
      float2 a = x[0], b = make_float2(0.f, 0.f);
      terms<K, 1>(p, q, a, b);
      // y_K = a -+ i b, y_{N-K} = a +- i b
      const float2 ib = INV ? make_float2(-b.y, b.x) : make_float2(b.y, -b.x);
      y[K] = make_float2(a.x + ib.x, a.y + ib.y);
      y[N - K] = make_float2(a.x - ib.x, a.y - ib.y);
      rows<K + 1>(x, p, q, y);
    }
  }
  template <int K, int M>
  static __device__ __forceinline__ void terms(const float2 (&p)[N / 2 + 1],
                                               const float2 (&q)[N / 2 + 1], float2 &a, float2 &b) {
    if constexpr (M <= N / 2) {
      constexpr float c = (float)turn(K * M, N, false), s = (float)turn(K * M, N, true);
      a = make_float2(fmaf(c, p[M].x, a.x), fmaf(c, p[M].y, a.y));
      b = make_float2(fmaf(s, q[M].x, b.x), fmaf(s, q[M].y, b.y));
      terms<K, M + 1>(p, q, a, b);
    }
  }
};

}  // namespace pm_dft
