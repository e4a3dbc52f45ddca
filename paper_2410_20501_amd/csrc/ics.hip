// Initial conditions by Lagrangian perturbation theory (paper Sect. 3.3 and App. A).
//
// pm_ic_lpt: the linear density at a = 1 from a white-noise grid and a P(k) table,
// DFT[delta] = sqrt(N) sqrt(P(k)) DFT[w] (unit box, N = n^3), with the k = 0 mode and
// the Nyquist planes zero; then, with every derivative taken in Fourier space,
//   Psi(1) = -grad phi(1),        phi(1) = lap^-1 delta
//   Psi(2) =  grad phi(2),        lap phi(2) = sum_{i<j} phi(1)_ii phi(1)_jj - phi(1)_ij^2
//   Psi(3a) = grad phi(3a),       lap phi(3a) = det phi(1)_ij
//   Psi(3b) = grad phi(3b),       lap phi(3b) = [tr phi(2)_ij tr phi(1)_ij
//                                                - phi(2)_ij phi(1)_ij] / 2
//   Psi(3c) = curl A(3c),         lap A(3c) = sum_i grad phi(2)_,i x grad phi(1)_,i
// and x = q + sum D^(k) Psi^(k), v = a^(1/2) sum k D^(k) Psi^(k) with the
// Einstein-de Sitter growth factors D = a, D2 = -3/7 D^2, D3a = -1/3 D^3,
// D3b = 10/21 D^3, D3c = -1/7 D^3. Products of fields are formed pointwise on a grid of
// m = n (dealias 0) or m = 2n (dealias 1: zero-padded spectra, free of aliasing for the
// quadratic and cubic terms) cells per side and truncated back to the band of the n grid.
//
// Everything is band limited: |m_d| < n/2 on every axis (the n grid's Nyquist planes are
// dropped). A spectrum is stored as its band, [n][n][Pb] with Pb = n/2 rounded up to 16
// (the rows of m_d = n/2 are ignored), and the transforms to and from the product grid
// take and leave only the band: the inverse passes along i, j, k start from n n/2 columns,
// m n/2 columns and m^2 rows. Wavenumber factors are constant along the other axes, so the
// six second derivatives need three transforms along i (of 1, k_x, k_x^2 times phi) and six
// along j; the k_z factors multiply the rows as they are read. At second order the rows of
// the six fields meet in registers, where their product is formed and transformed back: no
// field of the product grid goes to memory. At third order the twelve fields do (the
// products mix both Hessians). The displacements and the velocities are one vector
// transform each of the summed orders, written as whole particles with the lattice added.
//
// Bound by vector instructions and, above 128^3, by memory. Measured at second order with
// dealiasing, kernels of a call: 128^3 1236 -> 360 us, 256^3 3000 us; a 128^3 call 4911 -> 387
// us (two thirds of it were allocations, now kept: Scratch).
#include <cmath>
#include <new>
#include <vector>

#include "fft_line.h"

namespace {

using namespace pm_fft;

constexpr int kT = 256;
constexpr double kTwoPi = 6.283185307179586;

inline unsigned blocks_for(int64_t count, int threads) {
  return (unsigned)((count + threads - 1) / threads);
}

// log-log interpolation of the table, constant beyond its ends
__device__ double table_sqrt_p(double k, const double *__restrict__ lk, const double *__restrict__ lp,
                               int nt) {
  const double x = log(k);
  if (x <= lk[0]) return exp(0.5 * lp[0]);
  if (x >= lk[nt - 1]) return exp(0.5 * lp[nt - 1]);
  int lo = 0, hi = nt - 1;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (lk[mid] <= x) lo = mid;
    else hi = mid;
  }
  const double t = (x - lk[lo]) / (lk[hi] - lk[lo]);
  return exp(0.5 * (lp[lo] + t * (lp[hi] - lp[lo])));
}

// The place of a thread's column in a pass over 16-column tiles: line element t + N2 m.
template <int M>
struct Place {
  int c, t, o, kz, outer, base;
  __device__ __forceinline__ Place(int tiles) {
    using S = Split<M>;
    using C = ColShape<M>;
    c = threadIdx.x % kCols;
    const int u = threadIdx.x / kCols;
    t = u % S::N2;
    o = u / S::N2;
    const unsigned b = xcd_block(blockIdx.x, gridDim.x);
    kz = (int)(b % tiles) * kCols + c;
    outer = (int)(b / tiles) * C::OUT + o;
    base = o * C::LINE + c;
  }
};

// wavenumber of element e of a length-M axis and its place in the band of n (-1: outside)
template <int M>
__device__ __forceinline__ int signed_of(int e) {
  return e < M / 2 ? e : e - M;
}
__device__ __forceinline__ int band_of(int m, int n) {
  const int h = n / 2;
  return m > -h && m < h ? (m < 0 ? m + n : m) : -1;
}

__device__ __forceinline__ float power(float k, int p) { return p == 0 ? 1.0f : (p == 1 ? k : k * k); }

// sums of c[set][j] f[j] over the band spectra given
struct Combo {
  const float2 *f[4];
  double c[2][4];
  int count;
};

// 1 / m2 for an integer m2 > 0 (a Newton step on FP32's reciprocal), 0 for 0
__device__ __forceinline__ double inverse_of(int m2) {
  if (m2 == 0) return 0.0;
  const double r = (double)__builtin_amdgcn_rcpf((float)m2);
  return r * fma(-(double)m2, r, 2.0);
}

// sqrt(N P(k)) of every |m|^2 = t that the band holds (0 at 0): 3 (n/2)^2 logarithms and
// exponentials in FP64 instead of n^3 / 2 (128^3: the pass that applies them 28.6 -> 9.7 us and this one 4.7)
__global__ __launch_bounds__(kT) void k_amplitude(const double *__restrict__ lk,
                                                  const double *__restrict__ lp, int nt, float scale,
                                                  int count, float *__restrict__ amp) {
  const int t = blockIdx.x * kT + threadIdx.x;
  if (t < count) amp[t] = t ? (float)(scale * table_sqrt_p(kTwoPi * sqrt((double)t), lk, lp, nt)) : 0.0f;
}

// The k factors are formed from the integers m = k / (2 pi); the powers of 2 pi left over go
// into the weights. The factor c m_x^o / m^2 of a spectrum is formed in FP64 and rounded once;
// powers of m_y and m_z multiply later, one rounding each.

// Inverse along i: U = (sum of the spectra) (/ m^2 with DIV), then for o = 0 .. NOUT - 1
// out_o[i][ky][kz] = the transform of m_x^o U. With a grid of two in y, a second sum goes
// `set` values further on (the passes after it, likewise).
template <int M, int NOUT, bool DIV>
__global__ __launch_bounds__(ColShape<M>::NT) void k_band_inv_x(Combo in, float2 *o0, float2 *o1,
                                                                float2 *o2, int n, int Pb, size_t set,
                                                                const float2 *__restrict__ tw) {
  using S = Split<M>;
  __shared__ __align__(16) float lds[ColShape<M>::LDS];
  const Place<M> p(Pb / kCols);
  set *= blockIdx.y;
  const int my = p.outer < n / 2 ? p.outer : p.outer - n;
  const bool live = p.kz < n / 2 && p.outer != n / 2;
  const int yz = my * my + p.kz * p.kz;
  // U / c[0] (the other spectra by the ratio of their weights to the first's)
  const double c0 = in.c[blockIdx.y][0];
  float2 u[S::N1];
#pragma unroll
  for (int m = 0; m < S::N1; ++m) {
    const int mx = signed_of<M>(p.t + S::N2 * m), sx = band_of(mx, n);
    float2 v = make_float2(0.f, 0.f);
    if (live && sx >= 0) {
      const int64_t at = ((int64_t)sx * n + p.outer) * Pb + p.kz;
      v = in.f[0][at];
      for (int j = 1; j < in.count; ++j) {
        const float2 f = in.f[j][at];
        const float c = (float)(in.c[blockIdx.y][j] / c0);
        v = make_float2(fmaf(c, f.x, v.x), fmaf(c, f.y, v.y));
      }
    }
    u[m] = v;
  }
  float2 *out[3] = {o0, o1, o2};
#pragma unroll
  for (int o = 0; o < NOUT; ++o) {
    float2 x[S::N1];
#pragma unroll
    for (int m = 0; m < S::N1; ++m) {
      const int mx = signed_of<M>(p.t + S::N2 * m);
      const double w = DIV ? c0 * inverse_of(mx * mx + yz) : c0;
      const float f = (float)(w * (o == 0 ? 1 : (o == 1 ? mx : mx * mx)));
      x[m] = make_float2(f * u[m].x, f * u[m].y);
    }
    cols<M, true>(x, lds, p.base, p.t, tw);
    if (p.kz < n / 2)
#pragma unroll
      for (int m = 0; m < S::N1; ++m)
        out[o][set + ((size_t)(p.t + S::N2 * m) * n + p.outer) * Pb + p.kz] = x[m];
  }
}

// Inverse along j of the planes i = x0 .. : out_o[i - x0][j][kz] = the transform of m_y^o in.
// (On the n grid this pass and the three others along i and j have their columns in the same
// places before and after: a block reads its own whole before it writes, so an output may be
// the input.)
template <int M, int NOUT>
__global__ __launch_bounds__(ColShape<M>::NT) void k_band_inv_y(const float2 *in, float2 *o0,
                                                                float2 *o1, float2 *o2, int x0, int n,
                                                                int Pb, size_t set, const float2 *__restrict__ tw) {
  using S = Split<M>;
  __shared__ __align__(16) float lds[ColShape<M>::LDS];
  const Place<M> p(Pb / kCols);
  const bool live = p.kz < n / 2;
  set *= blockIdx.y;
  float2 u[S::N1];
#pragma unroll
  for (int m = 0; m < S::N1; ++m) {
    const int sy = band_of(signed_of<M>(p.t + S::N2 * m), n);
    u[m] = live && sy >= 0 ? in[set + ((size_t)(x0 + p.outer) * n + sy) * Pb + p.kz] : make_float2(0.f, 0.f);
  }
  float2 *out[3] = {o0, o1, o2};
#pragma unroll
  for (int o = 0; o < NOUT; ++o) {
    float2 x[S::N1];
#pragma unroll
    for (int m = 0; m < S::N1; ++m) {
      const float f = power((float)signed_of<M>(p.t + S::N2 * m), o);
      x[m] = make_float2(f * u[m].x, f * u[m].y);
    }
    cols<M, true>(x, lds, p.base, p.t, tw);
    if (live)
#pragma unroll
      for (int m = 0; m < S::N1; ++m)
        out[o][set + ((size_t)p.outer * M + p.t + S::N2 * m) * Pb + p.kz] = x[m];
  }
}

// Forward along j of the planes x0 .. : the band of the transform to out[i][ky][kz].
template <int M>
__global__ __launch_bounds__(ColShape<M>::NT) void k_band_fwd_y(const float2 *in, float2 *out, int x0, int n,
                                                                int Pb, const float2 *__restrict__ tw) {
  using S = Split<M>;
  __shared__ __align__(16) float lds[ColShape<M>::LDS];
  const Place<M> p(Pb / kCols);
  const bool live = p.kz < n / 2;
  float2 x[S::N1];
#pragma unroll
  for (int m = 0; m < S::N1; ++m)
    x[m] = live ? in[((int64_t)p.outer * M + p.t + S::N2 * m) * Pb + p.kz] : make_float2(0.f, 0.f);
  cols<M, false>(x, lds, p.base, p.t, tw);
#pragma unroll
  for (int m = 0; m < S::N1; ++m) {
    const int sy = band_of(signed_of<M>(p.t + S::N2 * m), n);
    if (live && sy >= 0) out[((int64_t)(x0 + p.outer) * n + sy) * Pb + p.kz] = x[m];
  }
}

// Forward along i: the band of the transform times scale or, with a table of them,
// the amplitude at |m|^2.
template <int M>
__global__ __launch_bounds__(ColShape<M>::NT) void k_band_fwd_x(const float2 *in, float2 *out, int n, int Pb,
                                                                float scale,
                                                                const float2 *__restrict__ tw,
                                                                const float *__restrict__ amp) {
  using S = Split<M>;
  __shared__ __align__(16) float lds[ColShape<M>::LDS];
  const Place<M> p(Pb / kCols);
  const bool live = p.kz < n / 2 && p.outer != n / 2;
  float2 x[S::N1];
#pragma unroll
  for (int m = 0; m < S::N1; ++m)
    x[m] = live ? in[((int64_t)(p.t + S::N2 * m) * n + p.outer) * Pb + p.kz] : make_float2(0.f, 0.f);
  cols<M, false>(x, lds, p.base, p.t, tw);
  const int my = p.outer < n / 2 ? p.outer : p.outer - n;
#pragma unroll
  for (int m = 0; m < S::N1; ++m) {
    const int mx = signed_of<M>(p.t + S::N2 * m), sx = band_of(mx, n);
    if (!live || sx < 0) continue;
    const float f = amp ? amp[mx * mx + my * my + p.kz * p.kz] : scale;
    out[((int64_t)sx * n + p.outer) * Pb + p.kz] = make_float2(f * x[m].x, f * x[m].y);
  }
}

// One row of a band spectrum (m_z < h), times m_z^kp and, with rot, times i: the packed line
// whose inverse DFT is the real row.
template <int L>
__device__ __forceinline__ void band_row(const float2 *__restrict__ s, int h, int kp, bool rot, int t,
                                         const float2 *__restrict__ tw, float2 (&v)[Split<L>::N1]) {
  using S = Split<L>;
  auto get = [&](int k) {
    if (k >= h) return make_float2(0.f, 0.f);
    const float f = power((float)k, kp);
    const float2 a = s[k];
    return rot ? make_float2(-f * a.y, f * a.x) : make_float2(f * a.x, f * a.y);
  };
#pragma unroll
  for (int m = 0; m < S::N1; ++m) {
    const int k = t + S::N2 * m;
    v[m] = real_join(get(k), get(L - k), tw[k]);
  }
}

// the band of a transformed row to memory
template <int L>
__device__ __forceinline__ void store_band(float2 *__restrict__ dst, int h, int t,
                                           const float2 (&v)[Split<L>::N1]) {
  using S = Split<L>;
#pragma unroll
  for (int m = 0; m < S::N1; ++m)
    if (t + S::N2 * m < h) dst[t + S::N2 * m] = v[m];
}

template <int L>
struct RowPlace {
  int t, r;
  int64_t row;
  __device__ __forceinline__ RowPlace() {
    t = threadIdx.x % Split<L>::N2;
    r = threadIdx.x / Split<L>::N2;
    row = (int64_t)xcd_block(blockIdx.x, gridDim.x) * RowShape<L>::R + r;
  }
};

// rows of a real grid -> band rows
template <int L>
__global__ __launch_bounds__(256) void k_rows_to_band(const float *__restrict__ x, float2 *__restrict__ out,
                                                      int64_t rows_n, int h, int Pb,
                                                      const float2 *__restrict__ tw) {
  using S = Split<L>;
  __shared__ float2 lds[RowShape<L>::LDS];
  const RowPlace<L> p;
  const bool live = p.row < rows_n;
  const float2 *src = reinterpret_cast<const float2 *>(x + (live ? p.row : 0) * 2 * L);
  float2 v[S::N1], last;
#pragma unroll
  for (int m = 0; m < S::N1; ++m) v[m] = src[p.t + S::N2 * m];
  real_forward<L>(v, last, lds + p.r * RowShape<L>::PITCH, p.t, tw);
  if (live) store_band<L>(out + p.row * Pb, h, p.t, v);
}

// band rows (times m_z^kp) -> rows of a real grid
template <int L>
__global__ __launch_bounds__(256) void k_band_to_rows(const float2 *__restrict__ in, float *__restrict__ x,
                                                      int64_t rows_n, int h, int Pb, int kp,
                                                      const float2 *__restrict__ tw) {
  using S = Split<L>;
  __shared__ float2 lds[RowShape<L>::LDS];
  const RowPlace<L> p;
  const bool live = p.row < rows_n;
  float2 v[S::N1];
  band_row<L>(in + (live ? p.row : 0) * Pb, h, kp, false, p.t, tw, v);
  rows<L, true>(v, lds + p.r * RowShape<L>::PITCH, p.t, tw, 2);
  if (!live) return;
  float2 *dst = reinterpret_cast<float2 *>(x + p.row * 2 * L);
#pragma unroll
  for (int m = 0; m < S::N1; ++m) dst[p.t + S::N2 * m] = v[m];
}

// The six second derivatives' band rows -> the band rows of the second-order source
// phi_xx (phi_yy + phi_zz) + phi_yy phi_zz - phi_xy^2 - phi_xz^2 - phi_yz^2. f: the fields
// xx, yy, zz, xy, xz, yz before their powers of m_z, `field` values apart; out may be the
// first of them (a block reads its rows whole before it writes them).
// A block takes 32 / N2 rows: 6 x 32 threads transform the six fields, then the first 32
// form the product and transform it back while the block's other waves have ended. Half
// its time is vector instructions (65 a value). Against one thread group per row that does
// the seven transforms in turn, which needs 256 registers (spills at lines of 512):
// 128^2 lines of 64: 17 (18) us, 128 256 lines of 128: 80 (74), 32 512 of 256: 72 (83).
template <int L>
struct SourceShape {
  using S = Split<L>;
  static constexpr int R = 32 / S::N2, NT = 6 * 32, LDS = 6 * R * RowShape<L>::PITCH;
};
template <int L>
__global__ __launch_bounds__(192) void k_rows_source2(const float2 *f, size_t field, float2 *out,
                                                      int64_t rows_n, int h, int Pb,
                                                      const float2 *__restrict__ tw) {
  using S = Split<L>;
  using B = SourceShape<L>;
  constexpr int PITCH = RowShape<L>::PITCH;
  __shared__ float2 lds[B::LDS];
  const int t = threadIdx.x % S::N2, l = threadIdx.x / S::N2, q = l / B::R, r = l % B::R;
  const int64_t row = (int64_t)xcd_block(blockIdx.x, gridDim.x) * B::R + r;
  const bool live = row < rows_n;
  float2 *line = lds + l * PITCH;
  float2 v[S::N1];
  band_row<L>(f + q * field + (size_t)(live ? row : 0) * Pb, h, q == 2 ? 2 : (q > 3 ? 1 : 0), false, t, tw,
              v);
  rows<L, true>(v, line, t, tw, 2);
  line_sync();
#pragma unroll
  for (int m = 0; m < S::N1; ++m) line[t + S::N2 * m] = v[m];
  __syncthreads();
  if (q) return;
#pragma unroll
  for (int m = 0; m < S::N1; ++m) {
    const float2 *e = line + t + S::N2 * m;
    const float2 xx = v[m], yy = e[B::R * PITCH], zz = e[2 * B::R * PITCH];
    const float2 xy = e[3 * B::R * PITCH], xz = e[4 * B::R * PITCH], yz = e[5 * B::R * PITCH];
    v[m] = make_float2(xx.x * (yy.x + zz.x) + yy.x * zz.x - xy.x * xy.x - xz.x * xz.x - yz.x * yz.x,
                       xx.y * (yy.y + zz.y) + yy.y * zz.y - xy.y * xy.y - xz.y * xz.y - yz.y * yz.y);
  }
  float2 last;
  real_forward<L>(v, last, line, t, tw);
  if (live) store_band<L>(out + row * Pb, h, t, v);
}

// The six distinct second derivatives of a potential, a[0..5] = xx, yy, zz, xy, xz, yz.
struct Hess {
  const float *a[6];
};

enum { kSrcS2 = 0, kSrcDet = 1, kSrcS3b = 2, kSrcRx = 3, kSrcRy = 4, kSrcRz = 5 };

// The pointwise sources of the higher orders (paper Sect. 3.3, explicit forms), from the
// second derivatives of phi(1) (A) and of phi(2) (B), for the cells from first on.
__global__ __launch_bounds__(kT) void k_lpt_source(Hess A, Hess B, int which, int64_t first, int64_t count,
                                                   float *__restrict__ out) {
  const int64_t o = (int64_t)blockIdx.x * kT + threadIdx.x, p = first + o;
  if (o >= count) return;
  const float axx = A.a[0][p], ayy = A.a[1][p], azz = A.a[2][p];
  const float axy = A.a[3][p], axz = A.a[4][p], ayz = A.a[5][p];
  float v = 0.0f;
  if (which == kSrcS2) {
    v = axx * (ayy + azz) + ayy * azz - axy * axy - axz * axz - ayz * ayz;
  } else if (which == kSrcDet) {
    v = axx * ayy * azz + 2.0f * axy * axz * ayz - ayz * ayz * axx - axz * axz * ayy -
        axy * axy * azz;
  } else {
    const float bxx = B.a[0][p], byy = B.a[1][p], bzz = B.a[2][p];
    const float bxy = B.a[3][p], bxz = B.a[4][p], byz = B.a[5][p];
    if (which == kSrcS3b)
      v = 0.5f * axx * (byy + bzz) + 0.5f * ayy * (bxx + bzz) + 0.5f * azz * (bxx + byy) -
          axy * bxy - axz * bxz - ayz * byz;
    else if (which == kSrcRx)
      v = bxy * axz - bxz * axy + ayz * (byy - bzz) - byz * (ayy - azz);
    else if (which == kSrcRy)
      v = byz * axy - bxy * ayz + axz * (bzz - bxx) - bxz * (azz - axx);
    else
      v = bxz * ayz - byz * axz + axy * (bxx - byy) - bxy * (axx - ayy);
  }
  out[o] = v;
}

// Third order: the vector spectrum i m_d (sum of the potentials' sources) / m^2 plus
// c (i m x R) / m^2, element by element over the band ([n][n][Pb]).
__global__ __launch_bounds__(kT) void k_vector_spectrum(Combo pot, const float2 *__restrict__ rx,
                                                        const float2 *__restrict__ ry,
                                                        const float2 *__restrict__ rz, float c, int n,
                                                        int Pb, float2 *__restrict__ ox,
                                                        float2 *__restrict__ oy, float2 *__restrict__ oz) {
  const int64_t at = (int64_t)blockIdx.x * kT + threadIdx.x;
  if (at >= (int64_t)n * n * Pb) return;
  const int kzi = (int)(at % Pb), iy = (int)(at / Pb % n), ix = (int)(at / ((int64_t)Pb * n));
  const int mx = ix < n / 2 ? ix : ix - n, my = iy < n / 2 ? iy : iy - n;
  if (kzi >= n / 2 || ix == n / 2 || iy == n / 2) return;
  const float kx = (float)mx, ky = (float)my, kz = (float)kzi;
  const int m2 = mx * mx + my * my + kzi * kzi;
  const float r = (float)inverse_of(m2);
  float2 s = make_float2(0.f, 0.f);
  for (int j = 0; j < pot.count; ++j) {
    const float2 f = pot.f[j][at];
    const float w = (float)pot.c[0][j];
    s = make_float2(fmaf(w, f.x, s.x), fmaf(w, f.y, s.y));
  }
  const float2 X = rx[at], Y = ry[at], Z = rz[at];
  auto put = [&](float2 *o, float k, float2 a, float ka, float2 b, float kb) {
    // i r [k s + c (ka a - kb b)]
    const float re = k * s.x + c * (ka * a.x - kb * b.x), im = k * s.y + c * (ka * a.y - kb * b.y);
    o[at] = make_float2(-r * im, r * re);
  };
  put(ox, kx, Z, ky, Y, kz);
  put(oy, ky, X, kz, Z, kx);
  put(oz, kz, Y, kx, X, ky);
}

// The three components' band rows -> particles, whole: with `rot` the rows are those of
// m_x phi, m_y phi and phi (times i, i and i m_z), else the vector's. pos != NULL: the
// lattice point plus the field, box units wrapped into [0, 1) or, with cell, the in-cell
// offset with the cell index carried; vel != NULL: vfac times the field. With a grid of two
// in y the first field gives the positions, the second the velocities.
template <int L>
__global__ __launch_bounds__(256) void k_rows_particles(const float2 *__restrict__ sx,
                                                        const float2 *__restrict__ sy,
                                                        const float2 *__restrict__ sz, bool rot, int Pb,
                                                        size_t set, const float2 *__restrict__ tw,
                                                        float *__restrict__ pos, int32_t *__restrict__ cell,
                                                        float *__restrict__ vel, float vfac) {
  using S = Split<L>;
  constexpr int n = 2 * L;
  __shared__ float2 lds[RowShape<L>::LDS];
  const RowPlace<L> p;
  const bool live = p.row < (int64_t)n * n;
  const size_t at = (size_t)(live ? p.row : 0) * Pb + blockIdx.y * set;
  if (gridDim.y == 2) {
    if (blockIdx.y == 0) vel = nullptr;
    else pos = nullptr;
  }
  float2 *line = lds + p.r * RowShape<L>::PITCH;
  float2 v[3][S::N1];
  band_row<L>(sx + at, L, 0, rot, p.t, tw, v[0]);
  band_row<L>(sy + at, L, 0, rot, p.t, tw, v[1]);
  band_row<L>(sz + at, L, rot ? 1 : 0, rot, p.t, tw, v[2]);
#pragma unroll
  for (int d = 0; d < 3; ++d) rows<L, true>(v[d], line, p.t, tw, 2);
  if (!live) return;
  const int i = (int)(p.row / n), j = (int)(p.row % n);
  const float fn = (float)n;
#pragma unroll
  for (int m = 0; m < S::N1; ++m) {
    const int k0 = 2 * (p.t + S::N2 * m);
    float f[2][3] = {{v[0][m].x, v[1][m].x, v[2][m].x}, {v[0][m].y, v[1][m].y, v[2][m].y}};
    const int64_t q = p.row * n + k0;
    if (vel) {
      Pair4 *dst = reinterpret_cast<Pair4 *>(vel + 3 * q);
      dst[0] = Pair4{vfac * f[0][0], vfac * f[0][1]};
      dst[1] = Pair4{vfac * f[0][2], vfac * f[1][0]};
      dst[2] = Pair4{vfac * f[1][1], vfac * f[1][2]};
    }
    if (!pos) continue;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const int ijk[3] = {i, j, k0 + e};
      int c[3];
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        if (!cell) {
          float x = ((float)ijk[d] + 0.5f) / fn + f[e][d];
          x -= floorf(x);
          f[e][d] = x >= 1.0f ? 0.0f : x;
        } else {
          const float s = fmaf(f[e][d], fn, 0.5f);
          float fl = floorf(s), o = s - fl;
          if (o >= 1.0f) {
            o = 0.0f;
            fl += 1.0f;
          }
          const int ci = (ijk[d] + (int)fl) % n;
          c[d] = ci < 0 ? ci + n : ci;
          f[e][d] = o;
        }
      }
      if (cell) cell[q + e] = (c[0] * n + c[1]) * n + c[2];
    }
    Pair4 *dst = reinterpret_cast<Pair4 *>(pos + 3 * q);
    dst[0] = Pair4{f[0][0], f[0][1]};
    dst[1] = Pair4{f[0][2], f[1][0]};
    dst[2] = Pair4{f[1][1], f[1][2]};
  }
}

// ------------------------------------------------------------------ launches by size

struct Grid {  // a transform size and the band it carries
  int n, Pb;
  const float2 *tw;
  hipStream_t s;
};

template <int M>
unsigned col_grid(const Grid &g, int outer) {
  return (unsigned)(g.Pb / kCols * (outer / ColShape<M>::OUT));
}
template <int M>
unsigned row_grid(int64_t rows_n) {
  return (unsigned)((rows_n + RowShape<M / 2>::R - 1) / RowShape<M / 2>::R);
}

// the passes of one transform size M as a table of launches
struct Passes {
  // (a NULL output: fewer of them)
  void (*inv_x)(const Grid &, const Combo &, float2 *, float2 *, float2 *, bool div, int sets);
  void (*inv_y)(const Grid &, const float2 *, float2 *, float2 *, float2 *, int x0, int planes, int sets);
  void (*fwd_y)(const Grid &, const float2 *, float2 *, int x0, int planes);
  void (*fwd_x)(const Grid &, const float2 *, float2 *, float, const float *amp);
  void (*to_band)(const Grid &, const float *, float2 *, int64_t rows_n);
  void (*to_rows)(const Grid &, const float2 *, float *, int64_t rows_n, int kp);
  void (*source2)(const Grid &, const float2 *, size_t field, float2 *, int64_t rows_n);
  void (*particles)(const Grid &, const float2 *, const float2 *, const float2 *, bool rot, float *,
                    int32_t *, float *, float, int sets);
};

template <int M>
struct Launch {
  static constexpr int NT = ColShape<M>::NT, L = M / 2;
  static void inv_x(const Grid &g, const Combo &in, float2 *o0, float2 *o1, float2 *o2, bool div, int sets) {
    const dim3 b(col_grid<M>(g, g.n), sets);
    const size_t set = (size_t)g.n * g.n * g.Pb;
    if (o2) k_band_inv_x<M, 3, true><<<b, NT, 0, g.s>>>(in, o0, o1, o2, g.n, g.Pb, set, g.tw);
    else if (o1) k_band_inv_x<M, 2, true><<<b, NT, 0, g.s>>>(in, o0, o1, o2, g.n, g.Pb, set, g.tw);
    else if (div) k_band_inv_x<M, 1, true><<<b, NT, 0, g.s>>>(in, o0, o1, o2, g.n, g.Pb, set, g.tw);
    else k_band_inv_x<M, 1, false><<<b, NT, 0, g.s>>>(in, o0, o1, o2, g.n, g.Pb, set, g.tw);
  }
  static void inv_y(const Grid &g, const float2 *in, float2 *o0, float2 *o1, float2 *o2, int x0, int planes,
                    int sets) {
    const dim3 b(col_grid<M>(g, planes), sets);
    const size_t set = (size_t)g.n * g.n * g.Pb;
    if (o2) k_band_inv_y<M, 3><<<b, NT, 0, g.s>>>(in, o0, o1, o2, x0, g.n, g.Pb, set, g.tw);
    else if (o1) k_band_inv_y<M, 2><<<b, NT, 0, g.s>>>(in, o0, o1, o2, x0, g.n, g.Pb, set, g.tw);
    else k_band_inv_y<M, 1><<<b, NT, 0, g.s>>>(in, o0, o1, o2, x0, g.n, g.Pb, set, g.tw);
  }
  static void fwd_y(const Grid &g, const float2 *in, float2 *out, int x0, int planes) {
    k_band_fwd_y<M><<<col_grid<M>(g, planes), NT, 0, g.s>>>(in, out, x0, g.n, g.Pb, g.tw);
  }
  static void fwd_x(const Grid &g, const float2 *in, float2 *out, float scale, const float *amp) {
    k_band_fwd_x<M><<<col_grid<M>(g, g.n), NT, 0, g.s>>>(in, out, g.n, g.Pb, scale, g.tw, amp);
  }
  static void to_band(const Grid &g, const float *x, float2 *out, int64_t rows_n) {
    k_rows_to_band<L><<<row_grid<M>(rows_n), 256, 0, g.s>>>(x, out, rows_n, g.n / 2, g.Pb, g.tw);
  }
  static void to_rows(const Grid &g, const float2 *in, float *x, int64_t rows_n, int kp) {
    k_band_to_rows<L><<<row_grid<M>(rows_n), 256, 0, g.s>>>(in, x, rows_n, g.n / 2, g.Pb, kp, g.tw);
  }
  static void source2(const Grid &g, const float2 *f, size_t field, float2 *out, int64_t rows_n) {
    const unsigned b = (unsigned)((rows_n + SourceShape<L>::R - 1) / SourceShape<L>::R);
    k_rows_source2<L><<<b, 192, 0, g.s>>>(f, field, out, rows_n, g.n / 2, g.Pb, g.tw);
  }
  static void particles(const Grid &g, const float2 *sx, const float2 *sy, const float2 *sz, bool rot,
                        float *pos, int32_t *cell, float *vel, float vfac, int sets) {
    const dim3 b(row_grid<M>((int64_t)M * M), sets);
    k_rows_particles<L><<<b, 256, 0, g.s>>>(sx, sy, sz, rot, g.Pb, (size_t)g.n * g.n * g.Pb, g.tw, pos, cell,
                                            vel, vfac);
  }
  static Passes table() { return {inv_x, inv_y, fwd_y, fwd_x, to_band, to_rows, source2, particles}; }
};

Passes passes_of(int m) {
  switch (m) {
    case 8: return Launch<8>::table();
    case 16: return Launch<16>::table();
    case 32: return Launch<32>::table();
    case 64: return Launch<64>::table();
    case 128: return Launch<128>::table();
    case 256: return Launch<256>::table();
    case 512: return Launch<512>::table();
    default: return Launch<1024>::table();
  }
}

// Device scratch of a call, one allocation carved up. A call takes the context's (which then
// has none) and gives it back for the next one if it is at most kKeep; a larger one is
// released before the call returns. (Twelve allocations and releases took two thirds of a
// 128^3 call.)
constexpr size_t kKeep = (size_t)2 << 30;

struct Scratch {
  pm_ctx *ctx;
  IcScratch *buf = nullptr;
  size_t used = 0;
  bool idle = false;  // the work that reads it is known to have ended
  template <class T>
  T *take(size_t count) {  // before open(): adds up the sizes
    T *p = buf ? reinterpret_cast<T *>((char *)buf->p + used) : nullptr;
    used += (count * sizeof(T) + 255) / 256 * 256;
    return p;
  }
  bool open() {
    buf = __atomic_exchange_n(&ctx->ic, (IcScratch *)nullptr, __ATOMIC_ACQ_REL);
    if (buf && buf->bytes < used) {
      ic_scratch_free(buf);
      buf = nullptr;
    }
    if (!buf) {
      void *p = nullptr;
      if (hipMalloc(&p, used) != hipSuccess) {
        (void)hipGetLastError();
        return false;
      }
      buf = new (std::nothrow) IcScratch{p, used};
      if (!buf) {
        (void)hipFree(p);
        return false;
      }
    }
    used = 0;
    return true;
  }
  ~Scratch() {
    if (!buf) return;
    if (!idle) (void)hipDeviceSynchronize();  // an early error return: queued work may read it
    IcScratch *none = nullptr;
    if (buf->bytes > kKeep ||
        !__atomic_compare_exchange_n(&ctx->ic, &none, buf, false, __ATOMIC_ACQ_REL, __ATOMIC_RELAXED))
      ic_scratch_free(buf);
  }
};

}  // namespace

void ic_scratch_free(IcScratch *b) {
  if (!b) return;
  (void)hipFree(b->p);
  delete b;
}

extern "C" {

int pm_ic_release(pm_ctx *ctx) {
  if (!ctx) return PM_ERR_ARG;
  ic_scratch_free(__atomic_exchange_n(&ctx->ic, (IcScratch *)nullptr, __ATOMIC_ACQ_REL));
  return PM_OK;
}

int pm_ic_lpt(pm_ctx *ctx, const float *noise, int ntab, const double *k_tab, const double *p_tab,
              int order, int dealias, double a0, float *pos, int32_t *cell, float *vel,
              pm_stream stream) {
  if (!ctx) return PM_ERR_ARG;
  if (!noise || !pos || !vel || !k_tab || !p_tab) return pm_fail(ctx, PM_ERR_ARG, "null pointer");
  if (order < 1 || order > 3) return pm_fail(ctx, PM_ERR_ARG, "order must be 1, 2 or 3");
  if (dealias != 0 && dealias != 1) return pm_fail(ctx, PM_ERR_ARG, "dealias must be 0 or 1");
  if (!(a0 > 0.0) || !std::isfinite(a0)) return pm_fail(ctx, PM_ERR_ARG, "scale factor must be > 0");
  if (ntab < 2 || ntab > 65536) return pm_fail(ctx, PM_ERR_ARG, "the P(k) table needs 2 .. 65536 points");
  std::vector<double> lt(2 * (size_t)ntab);
  for (int i = 0; i < ntab; ++i) {
    if (!(k_tab[i] > 0.0) || !(p_tab[i] > 0.0) || !std::isfinite(k_tab[i]) ||
        !std::isfinite(p_tab[i]) || (i > 0 && !(k_tab[i] > k_tab[i - 1])))
      return pm_fail(ctx, PM_ERR_ARG, "P(k) table: k ascending, k and P positive and finite");
    lt[i] = std::log(k_tab[i]);
    lt[ntab + i] = std::log(p_tab[i]);
  }
  const int n = ctx->n;
  const int m = dealias ? 2 * n : n;
  if ((n & (n - 1)) != 0 || m > 1024)
    return pm_fail(ctx, PM_ERR_SHAPE, "initial conditions need a power-of-two grid (2n <= 1024 "
                                      "with dealiasing)");
  const hipStream_t s = (hipStream_t)stream;
  const int64_t N = (int64_t)n * n * n, M = (int64_t)m * m * m;
  const int Pb = (n / 2 + 15) / 16 * 16;
  const size_t band = (size_t)n * n * Pb, half = (size_t)m * n * Pb, plane = (size_t)m * Pb;
  // planes of the product grid at a time: their six half-transformed fields stay cached
  // (at most 128 MiB), a multiple of the lines a workgroup takes together
  int chunk = m;
  while (chunk > 8 && 6 * plane * chunk * sizeof(float2) > ((size_t)128 << 20)) chunk /= 2;
  const int namp = 3 * (n / 2) * (n / 2);  // |m|^2 <= 3 (n/2 - 1)^2
  const size_t fields = 6 * plane * chunk;  // (complex values of the six half-transformed ones)
  Scratch sc{ctx};
  double *d_tab = nullptr;
  float2 *tw_n = nullptr, *tw_m = nullptr, *delta = nullptr, *src_sp[6] = {}, *nx[2] = {}, *ny[3] = {};
  float2 *mx[3] = {}, *my[6] = {}, *my2 = nullptr, *my3 = nullptr, *back = nullptr, *vec[3] = {};
  float *tab_n = nullptr, *tab_m = nullptr, *amp = nullptr, *h1[6] = {}, *h2[6] = {}, *tmp = nullptr;
  // Fields lie where others are no longer, or not yet, needed (bytes per cell of the n grid
  // without | with dealiasing on large grids: order 1 12, order 2 24 | 40, order 3 92 | 444,
  // and at most 128 MiB of half-transformed fields).
  for (int pass = 0; pass < 2; ++pass) {
    if (pass == 1 && !sc.open())
      return pm_fail(ctx, PM_ERR_NOMEM, "initial-condition scratch allocation failed");
    d_tab = sc.take<double>(2 * (size_t)ntab);
    tw_n = sc.take<float2>(n);
    tab_n = sc.take<float>(3 * n);
    amp = sc.take<float>(namp);
    delta = sc.take<float2>(order == 2 ? 2 * band : band);
    if (order == 1) {
      // the potential's passes in delta's place
      nx[0] = ny[2] = delta;
      nx[1] = ny[0] = sc.take<float2>(band);
      ny[1] = sc.take<float2>(band);
      continue;
    }
    tw_m = sc.take<float2>(m);
    tab_m = sc.take<float>(3 * m);
    float2 *const x3 = sc.take<float2>(order == 2 ? 4 * half : 3 * half);
    float2 *const sp = order == 2 ? nullptr : sc.take<float2>(6 * band + half);
    float *const h = order == 2 ? nullptr : sc.take<float>(12 * (size_t)M);
    size_t extra = order == 2 ? fields * sizeof(float2) : 0;  // bytes of what fits nowhere
    // first Hessian: over the second one; second: over the sources and the band returned to,
    // which come after it; sources: over the Hessian's first transforms
    const size_t source = plane * chunk * sizeof(float2) + (size_t)chunk * m * m * sizeof(float);
    const bool fit1 = fields * sizeof(float2) <= 6 * (size_t)M * sizeof(float);
    const bool fit2 = fields <= 5 * band + half, fit3 = source <= 3 * half * sizeof(float2);
    if (order == 3 && (!fit1 || !fit2)) extra = fields * sizeof(float2);
    if (order == 3 && !fit3) extra = std::max(extra, source);
    float2 *const rest = reinterpret_cast<float2 *>(sc.take<char>(extra));
    if (pass == 0) continue;
    for (int i = 0; i < 3; ++i) mx[i] = x3 + i * half;
    if (order == 2) {
      src_sp[0] = delta + band;
      back = x3 + 3 * half;
      my[0] = rest;
      nx[0] = ny[2] = x3;  // (two sets of each)
      nx[1] = ny[0] = x3 + 2 * band;
      ny[1] = delta;
    } else {
      for (int i = 0; i < 6; ++i) {
        src_sp[i] = sp + i * band;
        h1[i] = h + i * M;
        h2[i] = h + (6 + i) * M;
      }
      back = sp + 6 * band;
      my[0] = fit1 ? reinterpret_cast<float2 *>(h2[0]) : rest;
      my2 = fit2 ? src_sp[1] : rest;
      my3 = fit3 ? x3 : rest;
      tmp = reinterpret_cast<float *>(my3 + plane * chunk);
      for (int i = 0; i < 3; ++i) vec[i] = reinterpret_cast<float2 *>(h) + i * band;
    }
    for (int i = 1; i < 6; ++i) my[i] = my[0] + i * plane * chunk;
  }
  PM_HIP(ctx, hipMemcpyAsync(d_tab, lt.data(), sizeof(double) * 2 * ntab, hipMemcpyHostToDevice, s));
  const double *lk = d_tab, *lp = d_tab + ntab;
  PM_HIP(ctx, fft_tables(FftBufs{nullptr, nullptr, tw_n, tab_n}, n, 0, 0, s));
  if (order >= 2) PM_HIP(ctx, fft_tables(FftBufs{nullptr, nullptr, tw_m, tab_m}, m, 0, 0, s));
  const Grid gn{n, Pb, tw_n, s}, gm{n, Pb, tw_m, s};
  const Passes pn = passes_of(n), pm = passes_of(m);
  const double invN = 1.0 / (double)N;
  const float trunc = (float)((double)N / (double)M);  // DFT on the m grid -> n-grid units
  // linear density at a = 1: DFT[delta] = sqrt(N) sqrt(P) DFT[w]
  pn.to_band(gn, noise, delta, (int64_t)n * n);
  pn.fwd_y(gn, delta, delta, 0, n);
  k_amplitude<<<blocks_for(namp, kT), kT, 0, s>>>(lk, lp, ntab, (float)std::sqrt((double)N), namp, amp);
  pn.fwd_x(gn, delta, delta, 1.0f, amp);
  PM_HIP(ctx, hipGetLastError());
  // k_i k_j F / k^2 / N = m_i m_j F / m^2 / N of the band spectrum F, along i for all planes
  auto hessian_x = [&](const float2 *f) {
    pm.inv_x(gm, Combo{{f}, {{invN}}, 1}, mx[0], mx[1], mx[2], true, 1);
  };
  // ... and along j for planes x0 .. : xx, yy, zz, xy, xz, yz before their powers of m_z
  auto hessian_y = [&](int x0) {
    pm.inv_y(gm, mx[2], my[0], nullptr, nullptr, x0, chunk, 1);  // m_x^2
    pm.inv_y(gm, mx[1], my[4], my[3], nullptr, x0, chunk, 1);    // m_x, m_x m_y
    pm.inv_y(gm, mx[0], my[2], my[5], my[1], x0, chunk, 1);      // 1, m_y, m_y^2
  };
  static const int kz_power[6] = {0, 0, 2, 0, 1, 1};
  const int64_t crow = (int64_t)chunk * m;
  if (order >= 2) {
    // second-order source from phi(1)_ij = IDFT[k_i k_j delta / k^2] / N, a chunk of planes
    // at a time
    hessian_x(delta);
    for (int x0 = 0; x0 < m; x0 += chunk) {
      hessian_y(x0);
      if (order == 3)
        for (int c = 0; c < 6; ++c)
          pm.to_rows(gm, my[c], h1[c] + (int64_t)x0 * m * m, crow, kz_power[c]);
      pm.source2(gm, my[0], plane * chunk, my[0], crow);
      pm.fwd_y(gm, my[0], back, x0, chunk);
    }
    pm.fwd_x(gm, back, src_sp[0], trunc, nullptr);
    PM_HIP(ctx, hipGetLastError());
  }
  if (order == 3) {
    // phi(2)_ij = IDFT[k_i k_j S2 / k^2] / N, then the five third-order sources
    hessian_x(src_sp[0]);
    for (int i = 0; i < 6; ++i) my[i] = my2 + i * plane * chunk;
    for (int x0 = 0; x0 < m; x0 += chunk) {
      hessian_y(x0);
      for (int c = 0; c < 6; ++c) pm.to_rows(gm, my[c], h2[c] + (int64_t)x0 * m * m, crow, kz_power[c]);
    }
    const Hess A{{h1[0], h1[1], h1[2], h1[3], h1[4], h1[5]}};
    const Hess B{{h2[0], h2[1], h2[2], h2[3], h2[4], h2[5]}};
    for (int w = kSrcDet; w <= kSrcRz; ++w) {
      for (int x0 = 0; x0 < m; x0 += chunk) {
        k_lpt_source<<<blocks_for(crow * m, kT), kT, 0, s>>>(A, B, w, (int64_t)x0 * m * m, crow * m, tmp);
        pm.to_band(gm, tmp, my3, crow);
        pm.fwd_y(gm, my3, back, x0, chunk);
      }
      pm.fwd_x(gm, back, src_sp[w], trunc, nullptr);
    }
    PM_HIP(ctx, hipGetLastError());
  }
  // Psi(1)_d = IDFT[i k_d delta / k^2] / N, Psi(2)_d = IDFT[-i k_d S2 / k^2] / N, the same
  // for 3a and 3b, and Psi(3c)_d = IDFT[-i (k x R)_d / k^2] / N: displacements and
  // velocities weigh the orders differently (k_d / k^2 = m_d / (2 pi m^2))
  const double ra = std::sqrt(a0), w = 1.0 / (kTwoPi * (double)N);
  const double d2 = -3.0 / 7.0 * a0 * a0, d3a = -1.0 / 3.0 * a0 * a0 * a0, d3b = 10.0 / 21.0 * a0 * a0 * a0;
  const double d3c = -1.0 / 7.0 * a0 * a0 * a0;
  Combo pot{{delta, src_sp[0], src_sp[1], src_sp[2]}, {}, order == 3 ? 4 : order};
  for (int v = 0; v < 2; ++v) {  // displacements, velocities
    const double f = v ? ra : 1.0;
    pot.c[v][0] = f * a0 * w;
    pot.c[v][1] = -(v ? 2.0 : 1.0) * f * d2 * w;
    pot.c[v][2] = -(v ? 3.0 : 1.0) * f * d3a * w;
    pot.c[v][3] = -(v ? 3.0 : 1.0) * f * d3b * w;
  }
  if (order < 3) {
    // (at first order one is a multiple of the other)
    pn.inv_x(gn, pot, nx[0], nx[1], nullptr, true, order);
    pn.inv_y(gn, nx[1], ny[0], nullptr, nullptr, 0, n, order);  // m_x phi
    pn.inv_y(gn, nx[0], ny[2], ny[1], nullptr, 0, n, order);    // phi, m_y phi
    pn.particles(gn, ny[0], ny[1], ny[2], true, pos, cell, vel, order == 1 ? (float)ra : 1.0f, order);
  } else {
    for (int v = 0; v < 2; ++v) {
      const float c = (float)(-(v ? 3.0 * ra : 1.0) * d3c * w);
      for (int j = 0; j < 4; ++j) pot.c[0][j] = pot.c[v][j];
      k_vector_spectrum<<<blocks_for((int64_t)band, kT), kT, 0, s>>>(
          pot, src_sp[3], src_sp[4], src_sp[5], c, n, Pb, vec[0], vec[1], vec[2]);
      for (int d = 0; d < 3; ++d) {
        pn.inv_x(gn, Combo{{vec[d]}, {{1.0}}, 1}, vec[d], nullptr, nullptr, false, 1);
        pn.inv_y(gn, vec[d], vec[d], nullptr, nullptr, 0, n, 1);
      }
      pn.particles(gn, vec[0], vec[1], vec[2], false, v ? nullptr : pos, cell, v ? vel : nullptr, 1.0f, 1);
    }
  }
  PM_HIP(ctx, hipGetLastError());
  // (the table's host copy and a scratch above the kept size end with the call)
  PM_HIP(ctx, hipStreamSynchronize(s));
  sc.idle = true;
  return PM_OK;
}

}  // extern "C"
