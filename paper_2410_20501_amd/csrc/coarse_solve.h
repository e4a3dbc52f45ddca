// Coarsest multigrid level (8 to 18 cells a side, an even number), solved exactly by one
// workgroup (the recursion's last level, paper Sect. 3.7.1). On a periodic grid the
// seven-point operator is diagonal in the discrete Fourier basis:
//   L e^{i 2 pi (a i + b j + c k)/n} = lambda e^{...},
//   lambda = (s_a + s_b + s_c) / h^2,  s_m = 2 cos(2 pi m/n) - 2,
// so u = DFT^-1[ DFT[f] / lambda ] with the zero mode set to zero (the periodic
// problem's mean: the right-hand side's mean is dropped, the solution has mean zero).
//
// What bounds it is the chain of passes on one compute unit. A thread transforms whole
// lines in registers, with the length and every twiddle known at compile time; the k
// transform is real to half complex straight from global memory, the i transform is
// followed by its own inverse without leaving the registers, and the last k transform
// goes straight back, so the grid crosses LDS four times, as the n^2 (n/2 + 1) half
// spectrum.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "dft.h"

namespace pm_coarse {

constexpr int kThreads = 384;  // lines of the largest size: 18^2, whole waves
constexpr int kMaxN = 18;
constexpr int kSpec = kMaxN * kMaxN * (kMaxN / 2 + 1);  // complex values in LDS

using pm_dft::Dft;
using pm_dft::turn;

// Real line x[0 .. N) <-> half spectrum X[0 .. N/2] by a complex transform of half the
// length: z_m = x_{2m} + i x_{2m+1}, X_k = E_k + w^k O_k with E, O the even and odd parts
// of Z; the inverse forms (X_k + conj X_{N/2-k}) + i conj(w^k)(X_k - conj X_{N/2-k}) and
// gives N times the line.
template <int N, int K>
__device__ __forceinline__ void split(const float2 (&z)[N / 2], float2 (&X)[N / 2 + 1]) {
  if constexpr (K <= N / 2) {
    constexpr int a = K == N / 2 ? 0 : K, b = K == 0 ? 0 : N / 2 - K;
    constexpr float c = (float)turn(K, N, false), s = -(float)turn(K, N, true);
    const float2 E = make_float2(0.5f * (z[a].x + z[b].x), 0.5f * (z[a].y - z[b].y));
    const float2 O = make_float2(0.5f * (z[a].y + z[b].y), -0.5f * (z[a].x - z[b].x));
    X[K] = make_float2(E.x + (c * O.x - s * O.y), E.y + (c * O.y + s * O.x));
    split<N, K + 1>(z, X);
  }
}
template <int N, int K>
__device__ __forceinline__ void join(const float2 (&X)[N / 2 + 1], float2 (&z)[N / 2]) {
  if constexpr (K < N / 2) {
    constexpr float c = (float)turn(K, N, false), s = (float)turn(K, N, true);
    const float2 p = X[K], q = make_float2(X[N / 2 - K].x, -X[N / 2 - K].y);
    const float2 e = make_float2(p.x + q.x, p.y + q.y), d = make_float2(p.x - q.x, p.y - q.y);
    const float2 o = make_float2(c * d.x - s * d.y, c * d.y + s * d.x);
    z[K] = make_float2(e.x - o.y, e.y + o.x);
    join<N, K + 1>(X, z);
  }
}

// One pass over the half spectrum in LDS: the N-point transforms of lines of stride
// `stride` that start at `base`.
template <int N, bool INV>
__device__ __forceinline__ void line_pass(float2 *spec, int base, int stride) {
  float2 x[N];
#pragma unroll
  for (int m = 0; m < N; ++m) x[m] = spec[base + m * stride];
  Dft<N, INV, false>::run(x);
#pragma unroll
  for (int m = 0; m < N; ++m) spec[base + m * stride] = x[m];
}

// 1 / (s_a + rest), a = 0 .. N - 1 in registers of the i pass; the zero mode gives 0
template <int N, int A>
__device__ __forceinline__ void divide(float2 (&x)[N], float rest, float unit, bool zero) {
  if constexpr (A < N) {
    constexpr float sa = (float)(2.0 * turn(A, N, false) - 2.0);
    const float r = A == 0 && zero ? 0.0f : unit / (sa + rest);
    x[A] = make_float2(x[A].x * r, x[A].y * r);
    divide<N, A + 1>(x, rest, unit, zero);
  }
}

// s_m for a run-time m
template <int N>
__device__ __forceinline__ float symbol(int m) {
  float s = 0.0f;
  auto pick = [&](auto self, auto I) {
    constexpr int i = decltype(I)::value;
    if constexpr (i < N) {
      constexpr float v = (float)(2.0 * turn(i, N, false) - 2.0);
      s = m == i ? v : s;
      self(self, std::integral_constant<int, i + 1>{});
    }
  };
  pick(pick, std::integral_constant<int, 0>{});
  return s;
}

// ug = L^-1 (scale (fg - mean)) with zero mean on N^3 cells. spec: LDS, kSpec values.
template <int N>
__device__ __forceinline__ void solve(float *__restrict__ ug, const float *__restrict__ fg, float scale,
                                      float mean, float h2, float2 *spec) {
  constexpr int NH = N / 2 + 1;
  const int t = threadIdx.x;
  const bool row = t < N * N, line = t < N * NH;
  const int lo = t / NH, kz = t - lo * NH;  // a line of the j and i passes
  if (row) {
    const float2 *src = reinterpret_cast<const float2 *>(fg + (size_t)t * N);
    float2 z[N / 2], X[NH];
#pragma unroll
    for (int m = 0; m < N / 2; ++m) z[m] = src[m];
#pragma unroll
    for (int m = 0; m < N / 2; ++m)
      z[m] = make_float2(scale * (z[m].x - mean), scale * (z[m].y - mean));
    Dft<N / 2, false, false>::run(z);
    split<N, 0>(z, X);
#pragma unroll
    for (int k = 0; k < NH; ++k) spec[t * NH + k] = X[k];
  }
  __syncthreads();
  if (line) line_pass<N, false>(spec, lo * N * NH + kz, NH);
  __syncthreads();
  if (line) {
    // i transform, division by lambda (and by the transforms' N^3), inverse i transform
    float2 x[N];
    const int base = lo * NH + kz;
#pragma unroll
    for (int m = 0; m < N; ++m) x[m] = spec[base + m * N * NH];
    Dft<N, false, false>::run(x);
    divide<N, 0>(x, symbol<N>(lo) + symbol<N>(kz), h2 / (float)(N * N * N), lo == 0 && kz == 0);
    Dft<N, true, false>::run(x);
#pragma unroll
    for (int m = 0; m < N; ++m) spec[base + m * N * NH] = x[m];
  }
  __syncthreads();
  if (line) line_pass<N, true>(spec, lo * N * NH + kz, NH);
  __syncthreads();
  if (row) {
    float2 X[NH], z[N / 2];
#pragma unroll
    for (int k = 0; k < NH; ++k) X[k] = spec[t * NH + k];
    join<N, 0>(X, z);
    Dft<N / 2, true, false>::run(z);
    float2 *dst = reinterpret_cast<float2 *>(ug + (size_t)t * N);
#pragma unroll
    for (int m = 0; m < N / 2; ++m) dst[m] = z[m];
  }
}

// any coarsest size (uniform n)
__device__ __forceinline__ void solve_any(float *__restrict__ ug, const float *__restrict__ fg, float scale,
                                          float mean, int n, float h2, float2 *spec) {
  switch (n) {
    case 8: solve<8>(ug, fg, scale, mean, h2, spec); break;
    case 10: solve<10>(ug, fg, scale, mean, h2, spec); break;
    case 12: solve<12>(ug, fg, scale, mean, h2, spec); break;
    case 14: solve<14>(ug, fg, scale, mean, h2, spec); break;
    case 16: solve<16>(ug, fg, scale, mean, h2, spec); break;
    default: solve<18>(ug, fg, scale, mean, h2, spec); break;
  }
}

}  // namespace pm_coarse
