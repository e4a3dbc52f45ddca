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
// conjugate inverse (INV), unnormalised: even lengths split into the even and odd
// elements, odd lengths summed directly.
template <int N, bool INV>
struct Dft {
  static __device__ __forceinline__ void run(float2 (&x)[N]) {
    if constexpr (N == 2) {
      const float2 a = x[0], b = x[1];
      x[0] = make_float2(a.x + b.x, a.y + b.y);
      x[1] = make_float2(a.x - b.x, a.y - b.y);
    } else if constexpr (N % 2 == 0) {
      float2 e[N / 2], o[N / 2];
#pragma unroll
      for (int m = 0; m < N / 2; ++m) {
        e[m] = x[2 * m];
        o[m] = x[2 * m + 1];
      }
      Dft<N / 2, INV>::run(e);
      Dft<N / 2, INV>::run(o);
      combine<0>(x, e, o);
    } else {
      direct(x);
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
