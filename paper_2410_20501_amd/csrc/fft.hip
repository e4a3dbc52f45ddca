// FFT Poisson solvers of paper Sect. 3.8:
//   FFT      phi = IDFT[ G(k) DFT[rho] ], G = -coef / (k^2 W(k)^2), W = prod_d sinc(k_d h/2)^p;
//   FFT_7pt  the same with the seven-point eigenvalue (4/h^2) sum_d sin^2(k_d h/2) in place
//            of k^2 and no deconvolution;
//   FULL_FFT the force g = -grad phi taken in Fourier space, g_d = IDFT[-i k_d G DFT[rho]]
//            (Eq. exact_fullfft_kernel), with k_d = 0 on the Nyquist plane of axis d.
//
// Layout: the half spectrum is kept as complex float spec[i][j][kc],
// kc = 0 .. n/2, row pitch P (a multiple of the column-tile width).
// Five passes over memory, each a batch of 1D transforms in registers (fft_line.h):
//   A  rows along k, real -> half complex (length-n/2 complex FFT + split)
//   B  columns along j, forward
//   C  columns along i: forward, multiply by G, inverse (one kernel)
//   D  columns along j, inverse
//   E  rows along k, half complex -> real
// FULL_FFT: k_d is constant along the transforms of the other axes, so the force needs two
// spectra after C (the potential's and the i component's), three after D (the j component
// branches off the potential's), and E multiplies the k component as it reads it, the
// three rows of a cell transformed by one group of threads that writes whole (x, y, z)
// cells.
//
// The passes are bound by memory: one solve moves about 40 bytes a cell where 8 must move
// (a transform needs all of a line, and three axes do not fit a compute unit's LDS).
// Times are at fft_run.
#include <cmath>

#include "fft_line.h"

namespace {

using namespace pm_fft;

constexpr int kMaxN = 1024;

// the block's sum of nb partial sums over count cells -> the mean (every thread)
template <int NT>
__device__ __forceinline__ float mean_of(const double *__restrict__ partial, int nb, double count) {
  __shared__ double s_mean[NT / 64];
  double s = 0.0;
  for (int b = threadIdx.x; b < nb; b += NT) s += partial[b];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) s += __shfl_down(s, o, 64);
  if ((threadIdx.x & 63) == 0) s_mean[threadIdx.x >> 6] = s;
  __syncthreads();
  double t = 0.0;
#pragma unroll
  for (int w = 0; w < NT / 64; ++w) t += s_mean[w];
  return (float)(t / count);
}

// Where the mean of a real grid comes from: nowhere (it is not subtracted), a device
// value, or nb partial sums to add up.
struct Mean {
  const float *value;
  const double *partial;
  int nb;
};

// Pass A: each row x[0..n) -> X[0..n/2], n = 2 L.
// The mean of x is subtracted as it is read: the k = 0 mode is dropped by every kernel
// anyway, and a large mean would otherwise set the scale of the FP32 rounding of every
// other mode (a density of mean 1 with fluctuations of 0.3 loses about a factor 1 / 0.3 in
// relative accuracy at 512^3).
template <int L>
__global__ __launch_bounds__(256) void k_rows_r2c(const float *__restrict__ x, float2 *__restrict__ spec,
                                                  int P, const float2 *__restrict__ tw, Mean mean) {
  using S = Split<L>;
  using R = RowShape<L>;
  constexpr int n = 2 * L;
  __shared__ float2 lds[R::LDS];
  const int t = threadIdx.x % S::N2, r = threadIdx.x / S::N2;
  const int64_t row = (int64_t)xcd_block(blockIdx.x, gridDim.x) * R::R + r;
  const bool live = row < (int64_t)n * n;
  const float2 *src = reinterpret_cast<const float2 *>(x + (live ? row : 0) * n);
  float2 v[S::N1], last;
#pragma unroll
  for (int m = 0; m < S::N1; ++m) v[m] = src[t + S::N2 * m];
  const float mu = mean.partial ? mean_of<256>(mean.partial, mean.nb, (double)n * n * n)
                                : (mean.value ? *mean.value : 0.0f);
#pragma unroll
  for (int m = 0; m < S::N1; ++m) v[m] = make_float2(v[m].x - mu, v[m].y - mu);
  real_forward<L>(v, last, lds + r * R::PITCH, t, tw);
  if (!live) return;
  float2 *dst = spec + row * P;
#pragma unroll
  for (int m = 0; m < S::N1; ++m) dst[t + S::N2 * m] = v[m];
  if (t == 0) dst[L] = last;
}

// Pass E: X[0..n/2] -> x[0..n) (unnormalised: the 1/n^3 is in G).
template <int L>
__global__ __launch_bounds__(256) void k_rows_c2r(const float2 *__restrict__ spec, float *__restrict__ x,
                                                  int P, const float2 *__restrict__ tw) {
  using S = Split<L>;
  using R = RowShape<L>;
  constexpr int n = 2 * L;
  __shared__ float2 lds[R::LDS];
  const int t = threadIdx.x % S::N2, r = threadIdx.x / S::N2;
  const int64_t row = (int64_t)xcd_block(blockIdx.x, gridDim.x) * R::R + r;
  const bool live = row < (int64_t)n * n;
  const float2 *src = spec + (live ? row : 0) * P;
  float2 v[S::N1];
#pragma unroll
  for (int m = 0; m < S::N1; ++m) {
    const int k = t + S::N2 * m;
    v[m] = real_join(src[k], src[L - k], tw[k]);
  }
  rows<L, true>(v, lds + r * R::PITCH, t, tw, 2);
  if (!live) return;
  float2 *dst = reinterpret_cast<float2 *>(x + row * n);
#pragma unroll
  for (int m = 0; m < S::N1; ++m) dst[t + S::N2 * m] = v[m];
}

// Pass E of FULL_FFT: the three components of a row, from the spectra of the i and j
// components and of the potential (times -i k_z as it is read), written as whole cells.
template <int L>
__global__ __launch_bounds__(256) void k_rows_c2r3(const float2 *__restrict__ sx,
                                                   const float2 *__restrict__ sy,
                                                   const float2 *__restrict__ sp,
                                                   float *__restrict__ x, int P,
                                                   const float2 *__restrict__ tw,
                                                   const float *__restrict__ kv) {
  using S = Split<L>;
  using R = RowShape<L>;
  constexpr int n = 2 * L;
  __shared__ float2 lds[R::LDS];
  const int t = threadIdx.x % S::N2, r = threadIdx.x / S::N2;
  const int64_t row = (int64_t)xcd_block(blockIdx.x, gridDim.x) * R::R + r;
  const bool live = row < (int64_t)n * n;
  float2 v[3][S::N1];
  const float2 *src[3] = {sx, sy, sp};
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const float2 *s = src[d] + (live ? row : 0) * P;
#pragma unroll
    for (int m = 0; m < S::N1; ++m) {
      const int k = t + S::N2 * m;
      float2 a = s[k], b = s[L - k];
      if (d == 2) {
        const float ka = kv[k], kb = kv[L - k];
        a = make_float2(ka * a.y, -ka * a.x);
        b = make_float2(kb * b.y, -kb * b.x);
      }
      v[d][m] = real_join(a, b, tw[k]);
    }
  }
#pragma unroll
  for (int d = 0; d < 3; ++d) rows<L, true>(v[d], lds + r * R::PITCH, t, tw, 2);
  if (!live) return;
#pragma unroll
  for (int m = 0; m < S::N1; ++m) {
    Pair4 *dst = reinterpret_cast<Pair4 *>(x + (row * n + 2 * (t + S::N2 * m)) * 3);
    dst[0] = Pair4{v[0][m].x, v[1][m].x};
    dst[1] = Pair4{v[2][m].x, v[0][m].y};
    dst[2] = Pair4{v[1][m].y, v[2][m].y};
  }
}

// Passes B, C, D: transforms along j (AXIS 1) or i (AXIS 0) of tiles of 16 consecutive kc
// columns, from src to dst (the same buffer, or not). MODE:
//   0 forward; 1 forward, times G, inverse; 2 inverse;
//   3 forward, times G, inverse to dst and inverse of -i k_d times it to dst2;
//   4 inverse to dst and inverse of -i k_d times it to dst2 (d: this axis).
// G(mx, my, kz) = -scale / ((t0[mx] + t0[my] + t0[kz]) t1[mx] t1[my] t1[kz]) with the
// per-axis tables t0 = tab[0 .. n), t1 = tab[n .. 2n); k_d = tab[2n + m_d].
template <int N, int AXIS, int MODE>
__global__ __launch_bounds__(ColShape<N>::NT) void k_cols(const float2 *src, float2 *dst, float2 *dst2,
                                                          int P, const float2 *__restrict__ tw,
                                                          const float *__restrict__ tab, float scale) {
  using S = Split<N>;
  using C = ColShape<N>;
  __shared__ __align__(16) float lds[C::LDS];
  const int c = threadIdx.x % kCols, u = threadIdx.x / kCols, t = u % S::N2, o = u / S::N2;
  const unsigned b = xcd_block(blockIdx.x, gridDim.x);
  const unsigned tiles = N / 2 / kCols + 1;  // (the last tile holds the Nyquist column alone)
  const int kz = (int)(b % tiles) * kCols + c, outer = (int)(b / tiles) * C::OUT + o;
  const bool live = kz <= N / 2;
  const int base = o * C::LINE + c;
  const int64_t at = AXIS == 1 ? (int64_t)outer * N * P + kz : (int64_t)outer * P + kz;
  const int64_t step = AXIS == 1 ? P : (int64_t)N * P;
  float2 x[S::N1];
#pragma unroll
  for (int m = 0; m < S::N1; ++m)
    x[m] = live ? src[at + (t + S::N2 * m) * step] : make_float2(0.f, 0.f);
  if constexpr (MODE == 0 || MODE == 1 || MODE == 3) cols<N, false>(x, lds, base, t, tw);
  if constexpr (MODE == 1 || MODE == 3) {
    const float *t0 = tab, *t1 = tab + N;
    const int my = outer;
    const float a0 = t0[my] + t0[live ? kz : 0], a1 = t1[my] * t1[live ? kz : 0];
#pragma unroll
    for (int m = 0; m < S::N1; ++m) {
      const int mx = t + S::N2 * m;
      const float g = (mx | my | kz) != 0 ? -scale / ((t0[mx] + a0) * (t1[mx] * a1)) : 0.0f;
      x[m] = make_float2(x[m].x * g, x[m].y * g);
    }
  }
  if constexpr (MODE == 3 || MODE == 4) {
    const float *kv = tab + 2 * N;
    float2 y[S::N1];
#pragma unroll
    for (int m = 0; m < S::N1; ++m) {
      const float k = kv[t + S::N2 * m];
      y[m] = make_float2(k * x[m].y, -k * x[m].x);  // (-i k) x
    }
    cols<N, true>(y, lds, base, t, tw);
#pragma unroll
    for (int m = 0; m < S::N1; ++m)
      if (live) dst2[at + (t + S::N2 * m) * step] = y[m];
  }
  if constexpr (MODE != 0) cols<N, true>(x, lds, base, t, tw);
#pragma unroll
  for (int m = 0; m < S::N1; ++m)
    if (live) dst[at + (t + S::N2 * m) * step] = x[m];
}

// Twiddles tw[m] = e^{-2 pi i m / n} and the per-axis tables of the kernel, in FP64 on
// the device and rounded once. For wavenumber index i (m = i, or i - n above n/2):
//   kind 0 (Green's function with window deconvolution): t0 = k^2, k = 2 pi m (unit
//     box), t1 = sinc(omega/2)^(2 deconv), omega = k h = 2 pi m / n;
//   kind 1 (seven-point eigenvalue): t0 = (4 / h^2) sin^2(omega/2), t1 = 1;
//   kd = k, except 0 at the Nyquist index n/2 (the derivative of a self-conjugate mode).
__device__ void fill_tables(int i, float2 *__restrict__ tw, float *__restrict__ tab, int n, int deconv,
                            int kind) {
  double sn, cs;
  sincospi(-2.0 * (double)i / (double)n, &sn, &cs);
  tw[i] = make_float2((float)cs, (float)sn);
  const int m = i < n / 2 ? i : i - n;
  const double half = (double)m / (double)n;  // omega / (2 pi)
  const double sh = sinpi(half);
  if (kind == 1) {
    tab[i] = (float)(4.0 * (double)n * n * sh * sh);
    tab[n + i] = 1.0f;
  } else {
    const double k = 2.0 * M_PI * (double)m;
    const double sinc = (m == 0) ? 1.0 : sh / (M_PI * half);
    double w = 1.0;
    for (int p = 0; p < 2 * deconv; ++p) w *= sinc;
    tab[i] = (float)(k * k);
    tab[n + i] = (float)w;
  }
  tab[2 * n + i] = (i == n / 2) ? 0.0f : (float)(2.0 * M_PI * (double)m);
}

// The launch before the passes: the tables (the last blocks) and, with nb > 0, the partial
// sums of x over nb blocks in a fixed order.
__global__ __launch_bounds__(RED_THREADS) void k_fft_prepare(float2 *__restrict__ tw,
                                                             float *__restrict__ tab, int n, int deconv,
                                                             int kind, const float *__restrict__ x, int nb,
                                                             double *__restrict__ partial) {
  if ((int)blockIdx.x >= nb) {
    const int i = ((int)blockIdx.x - nb) * RED_THREADS + threadIdx.x;
    if (i < n) fill_tables(i, tw, tab, n, deconv, kind);
    return;
  }
  const int64_t pairs = (int64_t)n * n * n / 2, stride = (int64_t)nb * RED_THREADS;
  const float2 *x2 = reinterpret_cast<const float2 *>(x);
  double s = 0.0;
  int64_t i = (int64_t)blockIdx.x * RED_THREADS + threadIdx.x;
  for (; i + 3 * stride < pairs; i += 4 * stride) {
    const float2 a = x2[i], b = x2[i + stride], c = x2[i + 2 * stride], d = x2[i + 3 * stride];
    s += (((double)a.x + a.y) + ((double)b.x + b.y)) + (((double)c.x + c.y) + ((double)d.x + d.y));
  }
  for (; i < pairs; i += stride) s += (double)x2[i].x + x2[i].y;
  __shared__ double w[RED_THREADS / 64];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) s += __shfl_down(s, o, 64);
  if ((threadIdx.x & 63) == 0) w[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
    for (int q = 0; q < RED_THREADS / 64; ++q) t += w[q];
    partial[blockIdx.x] = t;
  }
}

// F::run<N>(...) for the grid size n
template <class F, class... A>
void by_size(int n, A... a) {
  switch (n) {
    case 8: F::template run<8>(a...); break;
    case 16: F::template run<16>(a...); break;
    case 32: F::template run<32>(a...); break;
    case 64: F::template run<64>(a...); break;
    case 128: F::template run<128>(a...); break;
    case 256: F::template run<256>(a...); break;
    case 512: F::template run<512>(a...); break;
    default: F::template run<kMaxN>(a...); break;
  }
}

template <int N>
unsigned row_blocks() {
  return (unsigned)(((int64_t)N * N + RowShape<N / 2>::R - 1) / RowShape<N / 2>::R);
}

template <int AXIS, int MODE>
struct Cols {
  template <int N>
  static void run(hipStream_t s, const FftBufs &b, const float2 *src, float2 *dst, float2 *dst2,
                  float scale) {
    using C = ColShape<N>;
    const unsigned blocks = (N / 2 / kCols + 1) * (N / C::OUT);
    k_cols<N, AXIS, MODE><<<blocks, C::NT, 0, s>>>(src, dst, dst2, fft_pitch_of(N), b.twiddle, b.tab, scale);
  }
};

struct Forward {  // pass A
  template <int N>
  static void run(hipStream_t s, const FftBufs &b, const float *x, Mean mean) {
    k_rows_r2c<N / 2><<<row_blocks<N>(), 256, 0, s>>>(x, b.spec, fft_pitch_of(N), b.twiddle, mean);
  }
};

struct Backward {  // pass E
  template <int N>
  static void run(hipStream_t s, const FftBufs &b, const float2 *spec, float *x) {
    k_rows_c2r<N / 2><<<row_blocks<N>(), 256, 0, s>>>(spec, x, fft_pitch_of(N), b.twiddle);
  }
};

struct Backward3 {
  template <int N>
  static void run(hipStream_t s, const FftBufs &b, const float2 *sx, const float2 *sy, const float2 *sp,
                  float *x) {
    k_rows_c2r3<N / 2><<<row_blocks<N>(), 256, 0, s>>>(sx, sy, sp, x, fft_pitch_of(N), b.twiddle,
                                                       b.tab + 2 * N);
  }
};

template <int AXIS, int MODE>
void run_cols(int n, hipStream_t s, const FftBufs &b, const float2 *src, float2 *dst, float2 *dst2,
              float scale) {
  by_size<Cols<AXIS, MODE>, hipStream_t, const FftBufs &, const float2 *, float2 *, float2 *, float>(
      n, s, b, src, dst, dst2, scale);
}

}  // namespace

int fft_pitch(int n) { return fft_pitch_of(n); }

size_t fft_spec_elems(int n) { return (size_t)n * n * fft_pitch(n); }

int fft_mean_blocks(int n) {
  return (int)std::min<int64_t>(RED_BLOCKS, ((int64_t)n * n * n / 2 + RED_THREADS - 1) / RED_THREADS);
}

// Us per solve on MI355X, with the LDS Stockham stages (registers at 256 only), a launch for
// the tables and two for the mean, and FULL_FFT's three separate inverse transforms, against
// these passes:
//        n      32          64         128        256        512
//   FFT       81 -> 27   84 -> 27   116 -> 42  243 -> 160  3291 -> 1489
//   FULL_FFT 177 -> 30  187 -> 34   232 -> 65  599 -> 329  8181 -> 3398
// (FULL_FFT moves 72 bytes a cell instead of 96, counted as the 40 of FFT are.)
hipError_t fft_run(const FftBufs &b, int n, const float *rho, const float *mean, double *partial,
                   float coef, int deconv, int kind, float *out, hipStream_t s) {
  const float scale = (float)((double)coef / ((double)n * n * n));
  float2 *spec = b.spec;
  const int nb = mean ? 0 : fft_mean_blocks(n);
  k_fft_prepare<<<nb + (n + RED_THREADS - 1) / RED_THREADS, RED_THREADS, 0, s>>>(
      b.twiddle, b.tab, n, deconv, kind == PM_FFT_7PT ? 1 : 0, rho, nb, partial);
  by_size<Forward, hipStream_t, const FftBufs &, const float *, Mean>(
      n, s, b, rho, Mean{mean, mean ? nullptr : partial, nb});
  run_cols<1, 0>(n, s, b, spec, spec, nullptr, scale);
  if (kind != PM_FFT_FULL) {
    run_cols<0, 1>(n, s, b, spec, spec, nullptr, scale);
    run_cols<1, 2>(n, s, b, spec, spec, nullptr, scale);
    by_size<Backward, hipStream_t, const FftBufs &, const float2 *, float *>(n, s, b, spec, out);
    return hipGetLastError();
  }
  // the force in Fourier space: the potential's spectrum in spec, the i and j components'
  // in spec2
  float2 *sx = b.spec2, *sy = b.spec2 + fft_spec_elems(n);
  run_cols<0, 3>(n, s, b, spec, spec, sx, scale);
  run_cols<1, 2>(n, s, b, sx, sx, nullptr, scale);
  run_cols<1, 4>(n, s, b, spec, spec, sy, scale);
  by_size<Backward3, hipStream_t, const FftBufs &, const float2 *, const float2 *, const float2 *, float *>(
      n, s, b, sx, sy, spec, out);
  return hipGetLastError();
}

hipError_t fft_tables(const FftBufs &b, int n, int deconv, int kind, hipStream_t s) {
  k_fft_prepare<<<(n + RED_THREADS - 1) / RED_THREADS, RED_THREADS, 0, s>>>(b.twiddle, b.tab, n, deconv, kind,
                                                                            nullptr, 0, nullptr);
  return hipGetLastError();
}

hipError_t fft_alloc(pm_ctx *ctx) {
  const int n = ctx->n;
  const size_t pitch = std::max(fft_pitch(n), spectrum_pitch(n));
  hipError_t e = hipMalloc(&ctx->twiddle, sizeof(float2) * n);
  if (e == hipSuccess) e = hipMalloc(&ctx->fft_tab, sizeof(float) * 3 * n);
  if (e == hipSuccess) e = hipMalloc(&ctx->spec, sizeof(float2) * n * n * pitch);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    if (ctx->twiddle) (void)hipFree(ctx->twiddle);
    if (ctx->fft_tab) (void)hipFree(ctx->fft_tab);
    ctx->twiddle = nullptr;
    ctx->fft_tab = nullptr;
    ctx->spec = nullptr;
  }
  return e;
}

int pm_fft_solve_kind(pm_ctx *ctx, const float *rho, float coef, int deconv, int kind, float *out,
                      hipStream_t s, const float *mean) {
  const int n = ctx->n;
  if (n < 8 || (n & (n - 1)) != 0)
    return pm_fail(ctx, PM_ERR_SHAPE, "FFT solver needs a power-of-two grid (8 .. 1024)");
  const size_t elems = fft_spec_elems(n);
  if (!ctx->spec && fft_alloc(ctx) != hipSuccess)
    return pm_fail(ctx, PM_ERR_NOMEM, "FFT scratch allocation failed");
  if (kind == PM_FFT_FULL && !ctx->spec2) {
    if (hipMalloc(&ctx->spec2, 2 * sizeof(float2) * elems) != hipSuccess) {
      ctx->spec2 = nullptr;
      return pm_fail(ctx, PM_ERR_NOMEM, "FFT scratch allocation failed");
    }
  }
  // (the mean of rho is subtracted before the transform: the one given, or summed first)
  FftBufs b{(float2 *)ctx->spec, (float2 *)ctx->spec2, ctx->twiddle, ctx->fft_tab};
  PM_HIP(ctx, fft_run(b, n, rho, mean, ctx->red_partial, coef, deconv, kind, out, s));
  return PM_OK;
}

int pm_fft_solve(pm_ctx *ctx, const float *rho, float coef, int deconv, float *phi, hipStream_t s,
                 const float *mean) {
  return pm_fft_solve_kind(ctx, rho, coef, deconv, PM_FFT_GREEN, phi, s, mean);
}
