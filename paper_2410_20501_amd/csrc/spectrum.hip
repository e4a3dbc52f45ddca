// Power-spectrum estimator (paper Sect. 4): P(k) of a density grid in shells of |k|.
//
// delta = rho / mean - 1, one mode's power |F|^2 / (N mean)^2 / W^2 with
// W = prod_d sinc(pi m_d / n)^deconv, weight 2 for 0 < kz < n/2 (the mode and its
// conjugate), shell b = rint(|m|) in 1 .. nbins; FP64 sums.
//
// The results are FP64 and follow the transform's rounding mode by mode, so the estimator
// keeps the transform it has always had (the butterflies of the FFT solvers are grouped
// differently, which moves a shell's power by 1e-8): rows along k, columns along j and
// along i, staged in LDS as Stockham radix-4 (+ one radix-2) stages, or, at n = 256, in
// registers. The i pass does not store its spectrum: its block bins the modes it holds.
//
// Binning mode by mode (window by pow and sin in FP64, three LDS atomics a mode with most
// lanes of a wave in one shell, then global atomics of every block into the same shells)
// took 208 of 400 us at 256^3; now 216 us in all (120 at 128^3 against 238, 2083 at 512^3
// against 3311, 18.8 ms at 1024^3 against 32.8), most of it the transform's passes.
#include <cmath>
#include <vector>

#include "fft_line.h"

namespace {

using pm_fft::cadd;
using pm_fft::cmul;
using pm_fft::conjf2;
using pm_fft::csub;

constexpr int FT = 256;   // threads per block
constexpr int TL = 4096;  // complex elements held in LDS per block
constexpr double kTwoPi = 6.283185307179586;
constexpr int kPkMaxBins = 1024;

template <int R>
__device__ __forceinline__ void butterfly(float2 *v) {
  if constexpr (R == 2) {
    const float2 a = v[0], b = v[1];
    v[0] = cadd(a, b);
    v[1] = csub(a, b);
  } else {
    const float2 a0 = cadd(v[0], v[2]), a1 = csub(v[0], v[2]);
    const float2 a2 = cadd(v[1], v[3]), d = csub(v[1], v[3]);
    const float2 a3 = make_float2(d.y, -d.x);  // d * (-i)
    v[0] = cadd(a0, a2);
    v[1] = cadd(a1, a3);
    v[2] = csub(a0, a2);
    v[3] = csub(a1, a3);
  }
}

// One Stockham stage on T independent length-L sequences in LDS.
// Element (col, idx) lives at col*L + idx (ROWS) or idx*T + col (!ROWS).
// Butterfly j of sub-transform size Ns: inputs x[j + r L/R], twiddle
// W_{Ns R}^{r (j mod Ns)}, outputs y[(j/Ns) Ns R + (j mod Ns) + r Ns].
template <int R, bool ROWS>
__device__ __forceinline__ void fft_stage(float2 *buf, int L, int T, int Ns, int logNs,
                                          const float2 *__restrict__ tw, int twstep) {
  constexpr int PER = TL / (R * FT);
  const int nb = L / R;
  float2 v[PER][R];
  int jj[PER], cc[PER];
#pragma unroll
  for (int b = 0; b < PER; ++b) {
    const int w = threadIdx.x + b * FT;
    int j, col;
    if constexpr (ROWS) {
      j = w % nb;
      col = w / nb;
    } else {
      col = w % T;
      j = w / T;
    }
    jj[b] = j;
    cc[b] = col;
#pragma unroll
    for (int r = 0; r < R; ++r) v[b][r] = buf[ROWS ? col * L + j + r * nb : (j + r * nb) * T + col];
  }
  __syncthreads();
  const int step = (L / (Ns * R)) * twstep;
#pragma unroll
  for (int b = 0; b < PER; ++b) {
    const int j = jj[b], col = cc[b];
    const int k = j & (Ns - 1);
#pragma unroll
    for (int r = 1; r < R; ++r) {
      float2 t = tw[r * k * step];
      v[b][r] = cmul(v[b][r], t);
    }
    butterfly<R>(v[b]);
    const int base = ((j >> logNs) << logNs) * R + k;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int o = base + r * Ns;
      buf[ROWS ? col * L + o : o * T + col] = v[b][r];
    }
  }
  __syncthreads();
}

template <bool ROWS>
__device__ void lds_fft(float2 *buf, int L, int T, const float2 *__restrict__ tw, int twstep) {
  int Ns = 1, logNs = 0;
  while (L / Ns >= 4) {
    fft_stage<4, ROWS>(buf, L, T, Ns, logNs, tw, twstep);
    Ns *= 4;
    logNs += 2;
  }
  if (Ns < L) fft_stage<2, ROWS>(buf, L, T, Ns, logNs, tw, twstep);
}

// Rows along k, real to half complex: z_m = x_{2m} + i x_{2m+1}, Z = FFT_{n/2}(z),
// E_k = (Z_k + conj Z_{n/2-k}) / 2, O_k = -i (Z_k - conj Z_{n/2-k}) / 2, X_k = E_k + w^k O_k.
__global__ __launch_bounds__(FT) void k_rows_r2c(const float *__restrict__ x,
                                                 float2 *__restrict__ spec, int n, int P,
                                                 const float2 *__restrict__ tw,
                                                 const float *__restrict__ mean) {
  __shared__ float2 buf[TL];
  const int L = n / 2, T = TL / L;
  const int64_t rows = (int64_t)n * n;
  const int64_t row0 = (int64_t)blockIdx.x * T;
  const float mu = mean ? *mean : 0.0f;
  for (int e = threadIdx.x; e < TL; e += FT) {
    const int col = e / L, m = e % L;
    const int64_t row = row0 + col;
    float2 v = make_float2(0.f, 0.f);
    if (row < rows) {
      v = reinterpret_cast<const float2 *>(x + row * n)[m];
      v.x -= mu;
      v.y -= mu;
    }
    buf[e] = v;
  }
  __syncthreads();
  lds_fft<true>(buf, L, T, tw, 2);
  for (int e = threadIdx.x; e < T * (L + 1); e += FT) {
    const int col = e / (L + 1), k = e % (L + 1);
    const int64_t row = row0 + col;
    if (row >= rows) continue;
    const float2 zk = buf[col * L + (k == L ? 0 : k)];
    const float2 zm = conjf2(buf[col * L + (k == 0 ? 0 : L - k)]);
    const float2 E = make_float2(0.5f * (zk.x + zm.x), 0.5f * (zk.y + zm.y));
    const float2 D = csub(zk, zm);
    const float2 O = make_float2(0.5f * D.y, -0.5f * D.x);  // -i D / 2
    spec[row * P + k] = cadd(E, cmul(tw[k], O));
  }
}

// 16-point DFT in registers, natural order in and out: a radix-4 pass over the four
// stride-4 subsequences, twiddles W_16^(n2 k1), a radix-4 pass across them.
__device__ __forceinline__ float2 w16(int m) {
  // e^{-2 pi i m / 16}, m = 0 .. 9
  constexpr float c[10] = {1.0f, 0.92387953251128674f, 0.70710678118654752f,
                           0.38268343236508977f, 0.0f, -0.38268343236508977f,
                           -0.70710678118654752f, -0.92387953251128674f, -1.0f,
                           -0.92387953251128674f};
  constexpr float sn[10] = {0.0f, 0.38268343236508977f, 0.70710678118654752f,
                            0.92387953251128674f, 1.0f, 0.92387953251128674f,
                            0.70710678118654752f, 0.38268343236508977f, 0.0f,
                            -0.38268343236508977f};
  return make_float2(c[m], -sn[m]);
}

__device__ __forceinline__ void dft16(float2 (&x)[16]) {
  float2 y[4][4];  // y[n2][k1]: DFT over n1 of x[4 n1 + n2]
#pragma unroll
  for (int n2 = 0; n2 < 4; ++n2) {
    float2 v[4] = {x[n2], x[4 + n2], x[8 + n2], x[12 + n2]};
    butterfly<4>(v);
#pragma unroll
    for (int k1 = 0; k1 < 4; ++k1) y[n2][k1] = (n2 * k1 == 0) ? v[k1] : cmul(v[k1], w16(n2 * k1));
  }
#pragma unroll
  for (int k1 = 0; k1 < 4; ++k1) {
    float2 v[4] = {y[0][k1], y[1][k1], y[2][k1], y[3][k1]};
    butterfly<4>(v);
#pragma unroll
    for (int k2 = 0; k2 < 4; ++k2) x[k1 + 4 * k2] = v[k2];
  }
}

constexpr int kC256Pad = 17;  // LDS row of 16 values plus one (bank spread)

// x: this thread's 16 inputs (elements j + 16 n1 of its column, in order of n1); out:
// elements j + 16 k2 of the transform (thread j of the column, c its column in the tile)
__device__ __forceinline__ void fft256_cols(float2 (&x)[16], float2 *lds, int c, int j,
                                            const float2 *__restrict__ tw) {
  dft16(x);  // x[k1] = DFT over n1 of the subsequence j
#pragma unroll
  for (int k1 = 1; k1 < 16; ++k1) {
    float2 t = tw[j * k1];
    x[k1] = cmul(x[k1], t);
  }
  __syncthreads();  // the previous transpose's reads are done
#pragma unroll
  for (int k1 = 0; k1 < 16; ++k1) lds[(c * 16 + k1) * kC256Pad + j] = x[k1];
  __syncthreads();
#pragma unroll
  for (int n2 = 0; n2 < 16; ++n2) x[n2] = lds[(c * 16 + j) * kC256Pad + n2];
  dft16(x);  // x[k2] = element j + 16 k2
}

// 8-point DFT in registers, natural order in and out (radix 4 over the two stride-2
// subsequences, twiddles W_8^(n2 k1), radix 2 across)
__device__ __forceinline__ void dft8(float2 (&x)[8]) {
  constexpr float h = 0.70710678118654752f;
  float2 v0[4] = {x[0], x[2], x[4], x[6]}, v1[4] = {x[1], x[3], x[5], x[7]};
  butterfly<4>(v0);
  butterfly<4>(v1);
  // W_8^k1 = e^{-i pi k1 / 4} for k1 = 1, 2, 3
  const float s = -1.0f;
  v1[1] = cmul(v1[1], make_float2(h, s * h));
  v1[2] = make_float2(-s * v1[2].y, s * v1[2].x);  // times (0, s)
  v1[3] = cmul(v1[3], make_float2(-h, s * h));
#pragma unroll
  for (int k1 = 0; k1 < 4; ++k1) {
    x[k1] = cadd(v0[k1], v1[k1]);
    x[k1 + 4] = csub(v0[k1], v1[k1]);
  }
}

// In-place length-128 transforms of the 32 rows of buf (row r at r * kRowPitch128,
// natural order in and out), as 16 x 8 four-step transforms: thread t = 0 .. 7 of a row
// takes the 16-point DFT of the stride-8 subsequence t, the twiddles W_128^(t k1), and
// after a transpose the two 8-point DFTs of k1 = t and t + 8. tw is the table of n = 256
// (W_128^m = tw[2 m]).
constexpr int kRowPitch128 = 132;  // 128 values plus 4 (spreads the rows over the banks)

__device__ __forceinline__ void fft128_rows(float2 *buf, const float2 *__restrict__ tw) {
  const int r = threadIdx.x >> 3, t = threadIdx.x & 7;
  float2 *row = buf + r * kRowPitch128;
  float2 x[16];
#pragma unroll
  for (int n1 = 0; n1 < 16; ++n1) x[n1] = row[8 * n1 + t];
  dft16(x);
#pragma unroll
  for (int k1 = 1; k1 < 16; ++k1) {
    float2 w = tw[2 * t * k1];
    x[k1] = cmul(x[k1], w);
  }
  __syncthreads();
#pragma unroll
  for (int k1 = 0; k1 < 16; ++k1) row[k1 * 8 + t] = x[k1];
  __syncthreads();
  float2 a[8], b[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    a[j] = row[t * 8 + j];
    b[j] = row[(t + 8) * 8 + j];
  }
  dft8(a);
  dft8(b);
  __syncthreads();
#pragma unroll
  for (int k2 = 0; k2 < 8; ++k2) {
    row[t + 16 * k2] = a[k2];
    row[t + 8 + 16 * k2] = b[k2];
  }
  __syncthreads();
}

// k_rows_r2c for n = 256 (32 rows per block) with the register transform
__global__ __launch_bounds__(FT) void k_rows_r2c256(const float *__restrict__ x,
                                                    float2 *__restrict__ spec, int P,
                                                    const float2 *__restrict__ tw,
                                                    const float *__restrict__ mean) {
  constexpr int n = 256, L = 128, T = 32;
  static_assert(FT == T * 8, "8 threads per row");
  __shared__ float2 buf[T * kRowPitch128];
  const int64_t rows = (int64_t)n * n;
  const int64_t row0 = (int64_t)blockIdx.x * T;
  const float mu = mean ? *mean : 0.0f;
  for (int e = threadIdx.x; e < T * L; e += FT) {
    const int col = e / L, m = e % L;
    const int64_t row = row0 + col;
    float2 v = make_float2(0.f, 0.f);
    if (row < rows) {
      v = reinterpret_cast<const float2 *>(x + row * n)[m];
      v.x -= mu;
      v.y -= mu;
    }
    buf[col * kRowPitch128 + m] = v;
  }
  __syncthreads();
  fft128_rows(buf, tw);
  for (int e = threadIdx.x; e < T * (L + 1); e += FT) {
    const int col = e / (L + 1), k = e % (L + 1);
    const int64_t row = row0 + col;
    if (row >= rows) continue;
    const float2 *b = buf + col * kRowPitch128;
    const float2 zk = b[k == L ? 0 : k];
    const float2 zm = conjf2(b[k == 0 ? 0 : L - k]);
    const float2 E = make_float2(0.5f * (zk.x + zm.x), 0.5f * (zk.y + zm.y));
    const float2 D = csub(zk, zm);
    const float2 O = make_float2(0.5f * D.y, -0.5f * D.x);  // -i D / 2
    spec[row * P + k] = cadd(E, cmul(tw[k], O));
  }
}


// Columns along j in place (n^2 / T tiles of T = TL / n columns).
__global__ __launch_bounds__(FT) void k_spectrum_cols(float2 *spec, int n, int P,
                                                      const float2 *__restrict__ tw) {
  __shared__ float2 buf[TL];
  const int T = TL / n, kc0 = blockIdx.x * T;
  float2 *plane = spec + (int64_t)blockIdx.y * n * P + kc0;
  for (int e = threadIdx.x; e < TL; e += FT) buf[e] = plane[(int64_t)(e / T) * P + e % T];
  __syncthreads();
  lds_fft<false>(buf, n, T, tw, 1);
  for (int e = threadIdx.x; e < TL; e += FT) plane[(int64_t)(e / T) * P + e % T] = buf[e];
}

__global__ __launch_bounds__(FT) void k_spectrum_cols256(float2 *spec, int P,
                                                         const float2 *__restrict__ tw) {
  constexpr int n = 256, T = 16;
  __shared__ float2 lds[T * 16 * kC256Pad];
  const int c = threadIdx.x & 15, j = threadIdx.x >> 4;
  float2 *col = spec + (int64_t)blockIdx.y * n * P + blockIdx.x * T + c;
  float2 x[16];
#pragma unroll
  for (int q = 0; q < 16; ++q) x[q] = col[(int64_t)(j + 16 * q) * P];
  fft256_cols(x, lds, c, j, tw);
#pragma unroll
  for (int q = 0; q < 16; ++q) col[(int64_t)(j + 16 * q) * P] = x[q];
}

// Shell sums of a block: power and |k| in FP64, modes as integers.
struct Shells {
  double p[kPkMaxBins], k[kPkMaxBins];
  unsigned c[kPkMaxBins];
};

// Adds the modes of a transformed tile (all mx, one my, columns kz0 .. kz0 + T - 1 of the
// half spectrum, element (mx, column) at buf[mx T + column]). A thread takes a pair
// mx, -mx (same |k|, same window) and eight consecutive kz, along which the shell changes
// once or twice: it adds to the shells in LDS when it does, so a mode costs a fifth of an
// atomic instead of three.
__device__ void bin_modes(const float2 *buf, int T, int kz0, int my, int n, int nbins, double norm,
                          const double *__restrict__ win, Shells &sh) {
  const int h = n / 2, segs = (T + 7) / 8, items = (h + 1) * segs;
  const double y2 = (double)my * my, wy = win[my < 0 ? my + n : my];
  for (int it = threadIdx.x; it < items; it += FT) {
    const int mx = it / segs, c0 = (it - mx * segs) * 8;
    const bool pair = mx > 0 && mx < h;
    const double xy = (double)mx * mx + y2, wxy = win[mx] * wy;
    int cur = -1;
    double sp = 0.0, sk = 0.0;
    unsigned sc = 0;
    for (int c = c0; c < min(c0 + 8, T); ++c) {
      const int iz = kz0 + c;
      if (iz > h) break;
      const double mm = sqrt(xy + (double)iz * iz);
      const int b = (int)rint(mm);
      if (b < 1 || b > nbins) continue;
      if (b != cur) {
        if (cur > 0) {
          atomicAdd(&sh.p[cur - 1], sp);
          atomicAdd(&sh.k[cur - 1], sk);
          atomicAdd(&sh.c[cur - 1], sc);
        }
        cur = b;
        sp = sk = 0.0;
        sc = 0;
      }
      const float2 v = buf[mx * T + c];
      double re = v.x * norm, im = v.y * norm;
      double pw = re * re + im * im;
      if (pair) {
        const float2 u = buf[(n - mx) * T + c];
        re = u.x * norm;
        im = u.y * norm;
        pw += re * re + im * im;
      }
      const double w = wxy * win[iz];
      const unsigned count = (iz == 0 || iz == h ? 1u : 2u) * (pair ? 2u : 1u);
      sp += (iz == 0 || iz == h ? 1.0 : 2.0) * (pw / (w * w));
      sk += (double)count * (kTwoPi * mm);
      sc += count;
    }
    if (cur > 0) {
      atomicAdd(&sh.p[cur - 1], sp);
      atomicAdd(&sh.k[cur - 1], sk);
      atomicAdd(&sh.c[cur - 1], sc);
    }
  }
}

__device__ __forceinline__ void clear_shells(Shells &sh, int nbins) {
  for (int b = threadIdx.x; b < nbins; b += FT) {
    sh.p[b] = sh.k[b] = 0.0;
    sh.c[b] = 0;
  }
}

// the block's sums to its rows of partial ([3 nbins][blocks])
__device__ __forceinline__ void store_shells(const Shells &sh, int nbins, double *__restrict__ partial) {
  __syncthreads();
  const int64_t nb = gridDim.x;
  for (int b = threadIdx.x; b < nbins; b += FT) {
    partial[(3 * b) * nb + blockIdx.x] = sh.p[b];
    partial[(3 * b + 1) * nb + blockIdx.x] = sh.k[b];
    partial[(3 * b + 2) * nb + blockIdx.x] = (double)sh.c[b];
  }
}

// Columns along i and their modes into the shells, tile after tile (the spectrum is not
// written back).
__global__ __launch_bounds__(FT) void k_spectrum_bins(const float2 *__restrict__ spec, int n, int P,
                                                      const float2 *__restrict__ tw,
                                                      const double *__restrict__ win,
                                                      const double *__restrict__ mean, int nbins,
                                                      double *__restrict__ partial) {
  __shared__ float2 buf[TL];
  __shared__ Shells sh;
  clear_shells(sh, nbins);
  const int T = TL / n, tiles = (n / 2) / T + 1;
  const double norm = 1.0 / ((double)n * n * n * mean[0]);
  for (int w = blockIdx.x; w < tiles * n; w += gridDim.x) {
    const int iy = w / tiles, kc0 = (w - iy * tiles) * T;
    __syncthreads();  // the previous tile's modes have been read
    for (int e = threadIdx.x; e < TL; e += FT)
      buf[e] = spec[((int64_t)(e / T) * n + iy) * P + kc0 + e % T];
    __syncthreads();
    lds_fft<false>(buf, n, T, tw, 1);
    bin_modes(buf, T, kc0, iy < n / 2 ? iy : iy - n, n, nbins, norm, win, sh);
  }
  store_shells(sh, nbins, partial);
}

__global__ __launch_bounds__(FT) void k_spectrum_bins256(const float2 *__restrict__ spec, int P,
                                                         const float2 *__restrict__ tw,
                                                         const double *__restrict__ win,
                                                         const double *__restrict__ mean, int nbins,
                                                         double *__restrict__ partial) {
  constexpr int n = 256, T = 16, tiles = n / 2 / T + 1;
  __shared__ float2 lds[T * 16 * kC256Pad];
  __shared__ Shells sh;
  clear_shells(sh, nbins);
  const int c = threadIdx.x & 15, j = threadIdx.x >> 4;
  const double norm = 1.0 / ((double)n * n * n * mean[0]);
  for (int w = blockIdx.x; w < tiles * n; w += gridDim.x) {
    const int iy = w / tiles, kc0 = (w - iy * tiles) * T;
    float2 x[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) x[q] = spec[((int64_t)(j + 16 * q) * n + iy) * P + kc0 + c];
    fft256_cols(x, lds, c, j, tw);  // (its first barrier follows the previous tile's modes)
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 16; ++q) lds[(j + 16 * q) * T + c] = x[q];
    __syncthreads();
    bin_modes(lds, T, kc0, iy < n / 2 ? iy : iy - n, n, nbins, norm, win, sh);
  }
  store_shells(sh, nbins, partial);
}

// out[e] = the sum of row e of partial ([rows][nb]), one wave per row
__global__ __launch_bounds__(FT) void k_spectrum_total(const double *__restrict__ partial, int rows, int nb,
                                                       double *__restrict__ out) {
  const int e = blockIdx.x * (FT / 64) + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  double s = 0.0;
  if (e < rows)
    for (int b = lane; b < nb; b += 64) s += partial[(int64_t)e * nb + b];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) s += __shfl_down(s, o, 64);
  if (e < rows && lane == 0) out[e] = s;
}

// Twiddles and the per-axis window sinc(pi m / n)^deconv of wavenumber index i, in FP64
// (twiddles rounded once).
__global__ void k_spectrum_tables(float2 *__restrict__ tw, double *__restrict__ win, int n, int deconv) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  double sn, cs;
  sincospi(-2.0 * (double)i / (double)n, &sn, &cs);
  tw[i] = make_float2((float)cs, (float)sn);
  const int m = i < n / 2 ? i : i - n;
  double w = 1.0;
  if (m != 0 && deconv > 0) {
    const double x = M_PI * m / n;
    w = pow(sin(x) / x, (double)deconv);
  }
  win[i] = w;
}

}  // namespace

// whole column tiles (TL / n columns)
int spectrum_pitch(int n) { return ((n / 2 + 1 + TL / n - 1) / (TL / n)) * (TL / n); }

extern "C" int pm_power_spectrum(pm_ctx *ctx, const float *rho, int deconv, int nbins, double *pk,
                      double *kmean, int64_t *nmodes, pm_stream stream) {
  if (!ctx) return PM_ERR_ARG;
  if (!rho || !pk) return pm_fail(ctx, PM_ERR_ARG, "null pointer");
  if (deconv < 0 || deconv > 3) return pm_fail(ctx, PM_ERR_ARG, "deconv must be 0 .. 3");
  if (nbins < 1 || nbins > kPkMaxBins) return pm_fail(ctx, PM_ERR_ARG, "nbins must be 1 .. 1024");
  const int n = ctx->n;
  if ((n & (n - 1)) != 0)
    return pm_fail(ctx, PM_ERR_SHAPE, "the power spectrum needs a power-of-two grid");
  const hipStream_t s = (hipStream_t)stream;
  const int64_t N = (int64_t)n * n * n;
  if (!ctx->spec && fft_alloc(ctx) != hipSuccess)
    return pm_fail(ctx, PM_ERR_NOMEM, "FFT scratch allocation failed");
  float2 *spec = (float2 *)ctx->spec, *tw = ctx->twiddle;
  const int P = spectrum_pitch(n), T = TL / n;
  // FP64 mean in red_result[2], FP32 mean (subtracted before the transform: a large mean
  // would set the scale of every mode's rounding) in mean_f[2]
  PM_HIP(ctx, launch_sum_moments(rho, N, ctx->red_partial, ctx->red_result, ctx->mean_f + 2, s));
  // the reduction scratch (3 x RED_PARTIAL_CAP doubles): window table, totals, and the block
  // sums where it holds those of all the workgroups; else (125 of them with 512 shells, half
  // a chip) they lie in the force grid, 3 n^3 floats of scratch. 512^3 with 256 shells 2708
  // -> 2072 us, 1024^3 with 512 35.2 -> 18.8 ms.
  double *win = ctx->red_partial, *total = win + 1024, *partial = total + 3 * kPkMaxBins;
  const int blocks = std::min(((n / 2) / T + 1) * n, 512);
  int64_t room = 3 * (int64_t)RED_PARTIAL_CAP - 1024 - 3 * kPkMaxBins;
  if (room < (int64_t)3 * nbins * blocks && 3 * N / 2 > room) {
    partial = reinterpret_cast<double *>(ctx->g);
    room = 3 * N / 2;
  }
  const int nb = (int)std::min<int64_t>(blocks, room / (3 * nbins));
  k_spectrum_tables<<<(n + 255) / 256, 256, 0, s>>>(tw, win, n, deconv);
  const unsigned rows = (unsigned)(((int64_t)n * n + TL / (n / 2) - 1) / (TL / (n / 2)));
  const dim3 cols(P / T, n);
  if (n == 256) {
    k_rows_r2c256<<<rows, FT, 0, s>>>(rho, spec, P, tw, ctx->mean_f + 2);
    k_spectrum_cols256<<<cols, FT, 0, s>>>(spec, P, tw);
    k_spectrum_bins256<<<nb, FT, 0, s>>>(spec, P, tw, win, ctx->red_result + 2, nbins, partial);
  } else {
    k_rows_r2c<<<rows, FT, 0, s>>>(rho, spec, n, P, tw, ctx->mean_f + 2);
    k_spectrum_cols<<<cols, FT, 0, s>>>(spec, n, P, tw);
    k_spectrum_bins<<<nb, FT, 0, s>>>(spec, n, P, tw, win, ctx->red_result + 2, nbins, partial);
  }
  k_spectrum_total<<<(3 * nbins + 3) / 4, FT, 0, s>>>(partial, 3 * nbins, nb, total);
  PM_HIP(ctx, hipGetLastError());
  std::vector<double> h(3 * (size_t)nbins);
  PM_HIP(ctx, hipMemcpyAsync(h.data(), total, sizeof(double) * 3 * nbins, hipMemcpyDeviceToHost, s));
  PM_HIP(ctx, hipStreamSynchronize(s));
  for (int b2 = 0; b2 < nbins; ++b2) {
    const double c = h[3 * b2 + 2];
    pk[b2] = c > 0.0 ? h[3 * b2] / c : 0.0;
    if (kmean) kmean[b2] = c > 0.0 ? h[3 * b2 + 1] / c : 0.0;
    if (nmodes) nmodes[b2] = (int64_t)std::llround(c);
  }
  return PM_OK;
}
