// Length-N transforms shared by a group of threads (device code of the FFT solvers and of
// the initial conditions).
//
// A line of N = N1 N2 values is held by N2 threads, thread t the elements t + N2 m,
// m = 0 .. N1 - 1. Four steps: N1-point DFTs over m in registers, twiddles W_N^(t k1), one
// exchange through LDS, then each thread's N1 / N2 transforms of length N2. The result is
// distributed like the input, so transforms chain without another exchange, and a pass
// with a multiplication between a forward and an inverse transform needs two.
#pragma once

#include "dft.h"
#include "internal.h"

namespace pm_fft {

__device__ __forceinline__ float2 cmul(float2 a, float2 b) {
  return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ float2 cadd(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ float2 csub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ float2 conjf2(float2 a) { return make_float2(a.x, -a.y); }

// N1 x N2 of a line: equal, or N1 = 2 N2
constexpr int first_of(int n) {
  int a = 1;
  while (a * a < n) a *= 2;
  return a;
}
template <int N>
struct Split {
  static constexpr int N1 = first_of(N), N2 = N / N1, Q = N1 / N2;
  static_assert(N1 * N2 == N && (Q == 1 || Q == 2), "power of two");
};

// Columns: 16 neighbouring columns side by side (c = 0 .. 15, consecutive lanes), so a
// load of one element of them is 128 contiguous bytes. A block takes kCols columns of OUT
// lines of the outer axis.
constexpr int kCols = 16;
template <int N>
struct ColShape {
  using S = Split<N>;
  static constexpr int NT = kCols * S::N2 > 256 ? kCols * S::N2 : 256;
  static constexpr int OUT = NT / (kCols * S::N2);
  // LDS row of one k1: N2 x 16 values and 16 more, which spreads the transposed reads over
  // the banks. Lines of 512 and more exchange real and imaginary parts one after the
  // other: half the LDS, twice the workgroups per compute unit.
  static constexpr int ROW = S::N2 * kCols + kCols, LINE = S::N1 * ROW;
  static constexpr bool HALVES = N >= 512;
  static constexpr int LDS = LINE * OUT * (HALVES ? 1 : 2);  // floats
};

template <int N, bool INV>
__device__ __forceinline__ void twiddle(float2 (&x)[Split<N>::N1], int t, const float2 *__restrict__ tw,
                                        int step) {
#pragma unroll
  for (int k = 1; k < Split<N>::N1; ++k) {
    float2 w = tw[t * k * step];
    if (INV) w.y = -w.y;
    x[k] = cmul(x[k], w);
  }
}

// the second DFTs of a line: y(h, n2) is this thread's element n2 of transform h
template <int N, bool INV>
__device__ __forceinline__ void second(float2 (&x)[Split<N>::N1]) {
  using S = Split<N>;
#pragma unroll
  for (int h = 0; h < S::Q; ++h) {
    float2 y[S::N2];
#pragma unroll
    for (int m = 0; m < S::N2; ++m) y[m] = x[h * S::N2 + m];
    pm_dft::Dft<S::N2, INV>::run(y);
#pragma unroll
    for (int m = 0; m < S::N2; ++m) x[h * S::N2 + m] = y[m];
  }
  if constexpr (S::Q == 2) {  // transform h's output k2 is element t + N2 (2 k2 + h)
    float2 z[S::N1];
#pragma unroll
    for (int m = 0; m < S::N1; ++m) z[m] = x[(m & 1) * S::N2 + (m >> 1)];
#pragma unroll
    for (int m = 0; m < S::N1; ++m) x[m] = z[m];
  }
}

// One transform of the block's columns, in place. lds: ColShape::LDS floats; t: the
// thread's place in its column (0 .. N2 - 1), base: its line's part of LDS plus its column.
template <int N, bool INV>
__device__ __forceinline__ void cols(float2 (&x)[Split<N>::N1], float *lds, int base, int t,
                                     const float2 *__restrict__ tw) {
  using S = Split<N>;
  using C = ColShape<N>;
  pm_dft::Dft<S::N1, INV>::run(x);
  twiddle<N, INV>(x, t, tw, 1);
  __syncthreads();  // the previous exchange's reads are done
  if constexpr (C::HALVES) {
#pragma unroll
    for (int part = 0; part < 2; ++part) {
      if (part) __syncthreads();
#pragma unroll
      for (int k = 0; k < S::N1; ++k) lds[base + k * C::ROW + t * kCols] = part ? x[k].y : x[k].x;
      __syncthreads();
#pragma unroll
      for (int h = 0; h < S::Q; ++h)
#pragma unroll
        for (int m = 0; m < S::N2; ++m) {
          const float v = lds[base + (t + h * S::N2) * C::ROW + m * kCols];
          if (part) x[h * S::N2 + m].y = v;
          else x[h * S::N2 + m].x = v;
        }
    }
  } else {
    float2 *l2 = reinterpret_cast<float2 *>(lds);
#pragma unroll
    for (int k = 0; k < S::N1; ++k) l2[base + k * C::ROW + t * kCols] = x[k];
    __syncthreads();
#pragma unroll
    for (int h = 0; h < S::Q; ++h)
#pragma unroll
      for (int m = 0; m < S::N2; ++m) x[h * S::N2 + m] = l2[base + (t + h * S::N2) * C::ROW + m * kCols];
  }
  second<N, INV>(x);
}

// Rows: N2 threads per line, 256 threads. LDS pitch of a line: at least N1 rows of N2 + 1
// values, and N2 modulo 32, so that neighbouring lines take neighbouring banks.
template <int N>
struct RowShape {
  using S = Split<N>;
  static constexpr int NT = 256, R = NT / S::N2;  // lines per block
  static constexpr int MIN = S::N1 * (S::N2 + 1);
  static constexpr int PITCH = MIN + ((S::N2 - MIN) % 32 + 32) % 32;
  static constexpr int LDS = R * PITCH;  // float2
};

// The threads of a line are N2 <= 16 neighbours, all of one wave, whose LDS accesses are
// performed in order: the exchange only has to keep the compiler from moving them.
__device__ __forceinline__ void line_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// one transform of the block's lines, in place (twiddles W_N^m = tw[m step])
template <int N, bool INV>
__device__ __forceinline__ void rows(float2 (&x)[Split<N>::N1], float2 *line, int t,
                                     const float2 *__restrict__ tw, int step) {
  using S = Split<N>;
  pm_dft::Dft<S::N1, INV>::run(x);
  twiddle<N, INV>(x, t, tw, step);
  line_sync();
#pragma unroll
  for (int k = 0; k < S::N1; ++k) line[k * (S::N2 + 1) + t] = x[k];
  line_sync();
#pragma unroll
  for (int h = 0; h < S::Q; ++h)
#pragma unroll
    for (int m = 0; m < S::N2; ++m) x[h * S::N2 + m] = line[(t + h * S::N2) * (S::N2 + 1) + m];
  second<N, INV>(x);
}

// Forward real line of n = 2 N values given as the packed z_m = x_{2m} + i x_{2m+1}: the
// half spectrum X_k of the thread's k = t + N2 m in x, and X_N (thread t = 0) in last.
// Z = DFT(z), X_k = E_k + w^k O_k, E = (Z_k + conj Z_{N-k}) / 2, O = -i (Z_k - conj Z_{N-k}) / 2.
template <int N>
__device__ __forceinline__ void real_forward(float2 (&x)[Split<N>::N1], float2 &last, float2 *line, int t,
                                             const float2 *__restrict__ tw) {
  using S = Split<N>;
  rows<N, false>(x, line, t, tw, 2);
  line_sync();
#pragma unroll
  for (int m = 0; m < S::N1; ++m) line[t + S::N2 * m] = x[m];
  line_sync();
  const float2 z0 = x[0];
#pragma unroll
  for (int m = 0; m < S::N1; ++m) {
    const int k = t + S::N2 * m;
    const float2 zk = x[m], zm = conjf2(line[k == 0 ? 0 : N - k]);
    const float2 E = make_float2(0.5f * (zk.x + zm.x), 0.5f * (zk.y + zm.y));
    const float2 D = csub(zk, zm);
    x[m] = cadd(E, cmul(tw[k], make_float2(0.5f * D.y, -0.5f * D.x)));
  }
  last = make_float2(z0.x - z0.y, 0.0f);
}

// Z~ of the inverse real transform from X_k and X_{N-k}: the inverse DFT of it gives
// 2 N (x_{2m} + i x_{2m+1})
__device__ __forceinline__ float2 real_join(float2 xk, float2 xnk, float2 w) {
  const float2 xm = conjf2(xnk);
  const float2 e = cadd(xk, xm), o = cmul(conjf2(w), csub(xk, xm));
  return make_float2(e.x - o.y, e.y + o.x);
}

}  // namespace pm_fft
