// Tile kernels of the linear multigrid's levels below the streaming ones (device code,
// shared by the single-box solver and the batched ensembles).
//
// These levels (a few thousand to a few million cells) fit the caches, so what bounds
// them is the number of dependent launches: with one kernel per half-sweep, residual,
// restriction and prolongation a V(2,2) visit of a level takes 11 launches of 3 to 7 us.
// Here a visit takes two. A workgroup owns a TI x TJ x TK tile of cells and loads it with
// a halo wide enough that every half-sweep can be recomputed for the halo as well
// (6 cells on the way down, 4 on the way up; the redundant work is cheap here):
//   tile_down  up to two red-black sweeps (red first), then the residual and its
//              restriction to the coarse grid; optionally the norms of the input's
//              residual (the convergence test of the cycle before)
//   tile_up    the trilinear prolongation of the coarse correction added as the tile is
//              loaded, then up to two sweeps (black first)
// Both are out of place: neighbouring tiles still read the old values of shared halos.
//
// A thread owns a pair of k-neighbouring columns (k even, k + 1) along i and keeps them,
// and their right-hand side, in registers: the i-neighbours cost nothing, and of the four
// in-plane neighbours one is the pair's other column. The other three come from LDS,
// where the columns are published by colour: E the column with j + k even, O the other
// one. Plane i of a half-sweep of colour c updates E when i + c is even, else O, so which
// array is read and which written is known at compile time, and one barrier separates
// two half-sweeps. Halo values are computed unmasked from whatever lies at the tile's
// edge: a wrong value moves one cell inward per half-sweep and never reaches the interior.
//
// Measured (MI355X), a V(2,2) cycle from a level down and back up, before and after:
//   32^3 (coarsest 16^3 included)  40 -> 17 us     64^3   78 -> 32 us
//   80^3                          123 -> 52 us    128^3  146 -> 71 us
// At 128^3 the two launches of the level take 25 + 17 us for 33.6 MB that must move (7 us
// at the card's copy rate): the halo's redundant updates (six times the interior's on the
// way down) keep the vector units and LDS busy. At 256^3 the streaming kernels, which
// recompute a halo along j and k only, are 1.5 times faster.
#pragma once

#include <hip/hip_runtime.h>

#include "internal.h"

namespace pm_tile {

// Shape of a tile kernel: interior TI x TJ x TK, halo H (all even).
template <int TI_, int TJ_, int TK_, int H_>
struct Shape {
  static constexpr int TI = TI_, TJ = TJ_, TK = TK_, H = H_;
  static constexpr int NI = TI + 2 * H, RJ = TJ + 2 * H, RK = TK + 2 * H, RK2 = RK / 2;
  static constexpr int NT = (RJ * RK2 + 63) / 64 * 64;  // threads (surplus ones work on padding)
  static constexpr int PAD = RK2 + 2;                   // read past the ends by edge threads
  static constexpr int ARR = NI * NT + 2 * PAD;         // floats of one colour array
  // the coarse correction's patch of tile_up, one coarse cell around the halved region
  static constexpr int CI = NI / 2 + 2, CJ = RJ / 2 + 2, CK = RK / 2 + 2;
  static constexpr int LDS = 2 * ARR, RAW = CI * CJ * CK;  // floats of LDS a tile works in
};
template <int TI, int TJ, int TK>
using Down = Shape<TI, TJ, TK, 6>;
template <int TI, int TJ, int TK>
using Up = Shape<TI, TJ, TK, 4>;

// One level's fields: the right-hand side is fscale (f - mean); the input iterate is
// uscale uin, or guess times the right-hand side where uin is NULL (the Jacobi step
// -h^2 / 6 that starts a coarse level, formed as it is needed instead of stored).
struct Level {
  const float *uin;
  float *uout;
  const float *f;
  float fscale, mean, uscale, guess;
  int n;
  float h2, inv_h2, omega;
};

// i mod n for -n <= i < 3 n (a tile reaches less than two periods past either end of a
// level of 18 cells or more, and of its coarse level)
__device__ __forceinline__ int wrap_near(int i, int n) {
  i += i < 0 ? n : 0;
  i -= i >= n ? n : 0;
  i -= i >= n ? n : 0;
  return i;
}

// the thread's pair of columns in the tile at (j0, k0)
template <class S>
struct Pair {
  int e;           // place in a plane of a colour array
  bool swp;        // E is the odd-k column
  int knE, knO;    // place of E's (O's) k-neighbour outside the pair
  unsigned col;    // offset of the even-k column in a plane
  bool inside;     // an interior pair of the grid
  int rj, r2;
  __device__ __forceinline__ Pair(int j0, int k0, int n) {
    const int t = threadIdx.x;
    rj = t / S::RK2;
    r2 = t - rj * S::RK2;
    const int gj = j0 - S::H + rj, gk = k0 - S::H + 2 * r2;  // gk even
    swp = (gj & 1) != 0;
    e = S::PAD + t;
    knE = swp ? e + 1 : e - 1;
    knO = swp ? e - 1 : e + 1;
    col = (unsigned)(wrap_near(gj, n) * n + wrap_near(gk, n));
    inside = rj >= S::H && rj < S::H + S::TJ && 2 * r2 >= S::H && 2 * r2 < S::H + S::TK && gj < n &&
             gk < n;
  }
};

template <class S>
struct Columns {
  float uE[S::NI], uO[S::NI], fE[S::NI], fO[S::NI];
};

// every load of the tile in flight, then the colours sorted out
template <class S>
__device__ __forceinline__ void load(const Level &a, const Pair<S> &p, int i0, Columns<S> &c) {
  const size_t nn = (size_t)a.n * a.n;
  int q = wrap_near(i0 - S::H, a.n);
  float2 u[S::NI], f[S::NI];
#pragma unroll
  for (int i = 0; i < S::NI; ++i) {
    const size_t at = (size_t)q * nn + p.col;
    f[i] = load_pair(a.f + at);
    if (a.uin) u[i] = load_pair(a.uin + at);
    q = q + 1 == a.n ? 0 : q + 1;
  }
#pragma unroll
  for (int i = 0; i < S::NI; ++i) {
    const float fx = a.fscale * (f[i].x - a.mean), fy = a.fscale * (f[i].y - a.mean);
    c.fE[i] = p.swp ? fy : fx;
    c.fO[i] = p.swp ? fx : fy;
    if (a.uin) {
      c.uE[i] = a.uscale * (p.swp ? u[i].y : u[i].x);
      c.uO[i] = a.uscale * (p.swp ? u[i].x : u[i].y);
    } else {
      c.uE[i] = a.guess * c.fE[i];
      c.uO[i] = a.guess * c.fO[i];
    }
  }
}

template <class S>
__device__ __forceinline__ void publish(const Pair<S> &p, const Columns<S> &c, float *LE, float *LO) {
#pragma unroll
  for (int i = 0; i < S::NI; ++i) {
    LE[p.e + i * S::NT] = c.uE[i];
    LO[p.e + i * S::NT] = c.uO[i];
  }
}

// Half-sweep number N (from 0) of colour C, on the planes that still matter after it.
template <class S, int N, int C, bool OM1>
__device__ __forceinline__ void half_sweep(const Level &a, const Pair<S> &p, Columns<S> &c, float *LE,
                                           float *LO) {
#pragma unroll
  for (int i = 1 + N; i < S::NI - 1 - N; ++i) {
    const int at = i * S::NT;
    if (((i + C) & 1) == 0) {
      const float nb = (LO[p.knE + at] + c.uO[i]) + (LO[p.e - S::RK2 + at] + LO[p.e + S::RK2 + at]) +
                       (c.uE[i - 1] + c.uE[i + 1]);
      const float gs = (nb - a.h2 * c.fE[i]) * (1.0f / 6.0f);
      c.uE[i] = OM1 ? gs : fmaf(a.omega, gs - c.uE[i], c.uE[i]);
      LE[p.e + at] = c.uE[i];
    } else {
      const float nb = (LE[p.knO + at] + c.uE[i]) + (LE[p.e - S::RK2 + at] + LE[p.e + S::RK2 + at]) +
                       (c.uO[i - 1] + c.uO[i + 1]);
      const float gs = (nb - a.h2 * c.fO[i]) * (1.0f / 6.0f);
      c.uO[i] = OM1 ? gs : fmaf(a.omega, gs - c.uO[i], c.uO[i]);
      LO[p.e + at] = c.uO[i];
    }
  }
  __syncthreads();
}

// hs half-sweeps (0, 2 or 4; uniform), the first of colour FIRST
template <class S, int FIRST, bool OM1>
__device__ __forceinline__ void sweeps(int hs, const Level &a, const Pair<S> &p, Columns<S> &c,
                                       float *LE, float *LO) {
  if (hs >= 2) {
    half_sweep<S, 0, FIRST, OM1>(a, p, c, LE, LO);
    half_sweep<S, 1, 1 - FIRST, OM1>(a, p, c, LE, LO);
  }
  if (hs >= 4) {
    half_sweep<S, 2, FIRST, OM1>(a, p, c, LE, LO);
    half_sweep<S, 3, 1 - FIRST, OM1>(a, p, c, LE, LO);
  }
}

// f - L u of the pair's two points on plane i, neighbours as published
template <class S>
__device__ __forceinline__ void residual(int i, const Level &a, const Pair<S> &p, const Columns<S> &c,
                                         const float *LE, const float *LO, float &rE, float &rO) {
  const int at = i * S::NT;
  const float x = c.uE[i], y = c.uO[i];
  // (sums of differences: exact for close values)
  const float lx = (LO[p.knE + at] - x) + (y - x) + (LO[p.e - S::RK2 + at] - x) +
                   (LO[p.e + S::RK2 + at] - x) + (c.uE[i - 1] - x) + (c.uE[i + 1] - x);
  const float ly = (LE[p.knO + at] - y) + (x - y) + (LE[p.e - S::RK2 + at] - y) +
                   (LE[p.e + S::RK2 + at] - y) + (c.uO[i - 1] - y) + (c.uO[i + 1] - y);
  rE = c.fE[i] - lx * a.inv_h2;
  rO = c.fO[i] - ly * a.inv_h2;
}

template <class S>
__device__ __forceinline__ void store(const Level &a, const Pair<S> &p, int i0, const Columns<S> &c) {
  if (!p.inside) return;
  const size_t nn = (size_t)a.n * a.n;
#pragma unroll
  for (int i = 0; i < S::TI; ++i)
    if (i0 + i < a.n) {
      const float x = c.uE[S::H + i], y = c.uO[S::H + i];
      *reinterpret_cast<Pair4 *>(a.uout + (size_t)(i0 + i) * nn + p.col) = p.swp ? Pair4{y, x} : Pair4{x, y};
    }
}

// hs half-sweeps on the tile at (i0, j0, k0), red first, and the restriction of the
// residual after them to fc (NULL: left out). NORM: sum[0..2] receive this thread's part
// of ||f - L u||^2 and ||f||^2 of the input and of the output's sum over the tile's interior.
template <int TI, int TJ, int TK, int KIND, bool OM1, bool NORM>
__device__ __forceinline__ void tile_down(const Level &a, int i0, int j0, int k0, int hs,
                                          float *__restrict__ fc, float *lds, double (&sum)[3]) {
  using S = Down<TI, TJ, TK>;
  const Pair<S> p(j0, k0, a.n);
  Columns<S> c;
  float *LE = lds, *LO = lds + S::ARR;
  load<S>(a, p, i0, c);
  publish<S>(p, c, LE, LO);
  __syncthreads();
  if constexpr (NORM) {
    sum[0] = sum[1] = sum[2] = 0.0;
#pragma unroll
    for (int i = S::H; i < S::H + S::TI; ++i) {
      float rE, rO;
      residual<S>(i, a, p, c, LE, LO, rE, rO);
      if (p.inside && i0 + i - S::H < a.n) {
        // (squared in FP64: a source of any size, a cotangent among them, keeps its norm; a
        // solve takes as long as with FP32 squares, 128^3 658 against 657 us)
        const double a64 = rE, b64 = rO, f64 = c.fE[i], g64 = c.fO[i];
        sum[0] += fma(a64, a64, b64 * b64);
        sum[1] += fma(f64, f64, g64 * g64);
      }
    }
    __syncthreads();  // every read of the input's values precedes the first update
  }
  sweeps<S, 0, OM1>(hs, a, p, c, LE, LO);
  store<S>(a, p, i0, c);
  if constexpr (NORM) {
#pragma unroll
    for (int i = S::H; i < S::H + S::TI; ++i)
      if (p.inside && i0 + i - S::H < a.n) sum[2] += (double)c.uE[i] + (double)c.uO[i];
  }
  if (!fc) return;
  // weights along i in registers: one value per coarse plane and column
  float cE[S::TI / 2], cO[S::TI / 2];
#pragma unroll
  for (int I = 0; I < S::TI / 2; ++I) cE[I] = cO[I] = 0.0f;
#pragma unroll
  for (int i = S::H - 1; i <= S::H + S::TI; ++i) {
    float rE, rO;
    residual<S>(i, a, p, c, LE, LO, rE, rO);
    const int d = i - S::H;  // fine plane within the tile, -1 .. TI
#pragma unroll
    for (int I = 0; I < S::TI / 2; ++I) {
      const int o = d - 2 * I;  // -1 .. 2: the four planes of a full-weighting stencil
      const float w = KIND == PM_RESTRICT_FW ? ((o == 0 || o == 1) ? 3.0f : 1.0f) : 1.0f;
      const bool takes = KIND == PM_RESTRICT_FW ? (o >= -1 && o <= 2) : (o == 0 || o == 1);
      if (takes) {
        cE[I] = fmaf(w, rE, cE[I]);
        cO[I] = fmaf(w, rO, cO[I]);
      }
    }
  }
  __syncthreads();  // the columns' last reads: their LDS takes the planes (rows of RK values)
  constexpr int PL = S::NT * 2;  // floats of one plane
#pragma unroll
  for (int I = 0; I < S::TI / 2; ++I)
    *reinterpret_cast<float2 *>(lds + I * PL + 2 * (int)threadIdx.x) =
        p.swp ? make_float2(cO[I], cE[I]) : make_float2(cE[I], cO[I]);
  __syncthreads();
  constexpr int HJ = S::TJ / 2, HK = S::TK / 2, CELLS = S::TI / 2 * HJ * HK;
  const int nc = a.n >> 1;
  for (int t = threadIdx.x; t < CELLS; t += S::NT) {
    const int I = t / (HJ * HK), J = t / HK % HJ, K = t % HK;
    float s = 0.0f;
    if constexpr (KIND == PM_RESTRICT_FW) {
      const float *r = lds + I * PL + (2 * J + S::H - 1) * S::RK + 2 * K + S::H - 1;
#pragma unroll
      for (int b = 0; b < 4; ++b, r += S::RK)
        s = fmaf(b == 0 || b == 3 ? 1.0f : 3.0f, (r[0] + r[3]) + 3.0f * (r[1] + r[2]), s);
      s *= 1.0f / 512.0f;
    } else {
      const float *r = lds + I * PL + (2 * J + S::H) * S::RK + 2 * K + S::H;
      s = 0.125f * ((r[0] + r[1]) + (r[S::RK] + r[S::RK + 1]));
    }
    const int gi = i0 / 2 + I, gj = j0 / 2 + J, gk = k0 / 2 + K;
    if (gi < nc && gj < nc && gk < nc) fc[((size_t)gi * nc + gj) * nc + gk] = s;
  }
}

// u + P ec on the tile at (i0, j0, k0) (ec NULL: u), then hs half-sweeps, black first.
// lds: LDS floats of the tile, raw: RAW floats for the coarse patch.
template <int TI, int TJ, int TK, bool OM1>
__device__ __forceinline__ void tile_up(const Level &a, const float *__restrict__ ec, int i0, int j0,
                                        int k0, int hs, float *lds, float *raw) {
  using S = Up<TI, TJ, TK>;
  const Pair<S> p(j0, k0, a.n);
  Columns<S> c;
  float *LE = lds, *LO = lds + S::ARR;
  // the coarse patch, one cell more on each side than the halved region: its loads are in
  // flight before the tile's own
  constexpr int N = S::RAW, PER = (N + S::NT - 1) / S::NT;
  float patch[PER];
  if (ec) {
    const int nc = a.n >> 1;
    const int I0 = (i0 - S::H) / 2 - 1, J0 = (j0 - S::H) / 2 - 1, K0 = (k0 - S::H) / 2 - 1;
#pragma unroll
    for (int m = 0; m < PER; ++m) {
      const int t = min((int)threadIdx.x + m * S::NT, N - 1);  // surplus: the last one again
      const int I = t / (S::CJ * S::CK), r = t - I * (S::CJ * S::CK), J = r / S::CK, K = r - J * S::CK;
      patch[m] = ec[((size_t)wrap_near(I0 + I, nc) * nc + wrap_near(J0 + J, nc)) * nc +
                    wrap_near(K0 + K, nc)];
    }
  }
  load<S>(a, p, i0, c);
  if (ec) {
#pragma unroll
    for (int m = 0; m < PER; ++m) {
      const int t = (int)threadIdx.x + m * S::NT;
      if (t < N) raw[t] = patch[m];
    }
    __syncthreads();
    // fine j takes 3/4 of coarse row J and 1/4 of the one on its side; the pair's columns
    // 2K, 2K + 1 take K - 1, K and K, K + 1 (surplus threads stay within the patch)
    const int jr = min(p.rj / 2 + 1, S::CJ - 2), jf = jr + ((p.rj & 1) ? 1 : -1);
    const float *near = raw + jr * S::CK + p.r2, *far = raw + jf * S::CK + p.r2;
    float ev[S::CI], od[S::CI];
#pragma unroll
    for (int I = 0; I < S::CI; ++I) {
      const int at = I * (S::CJ * S::CK);
      const float m = fmaf(0.75f, near[at], 0.25f * far[at]);
      const float z = fmaf(0.75f, near[at + 1], 0.25f * far[at + 1]);
      const float q = fmaf(0.75f, near[at + 2], 0.25f * far[at + 2]);
      ev[I] = fmaf(0.75f, z, 0.25f * m);
      od[I] = fmaf(0.75f, z, 0.25f * q);
    }
#pragma unroll
    for (int i = 0; i < S::NI; ++i) {
      const int A = i / 2 + 1, B = (i & 1) ? A + 1 : A - 1;
      const float e = fmaf(0.75f, ev[A], 0.25f * ev[B]), o = fmaf(0.75f, od[A], 0.25f * od[B]);
      c.uE[i] += p.swp ? o : e;
      c.uO[i] += p.swp ? e : o;
    }
  }
  if (hs > 0) {
    publish<S>(p, c, LE, LO);
    __syncthreads();
    sweeps<S, 1, OM1>(hs, a, p, c, LE, LO);
  }
  store<S>(a, p, i0, c);
}

// tiles of a level along one axis
__host__ __device__ inline int tiles_of(int n, int t) { return (n + t - 1) / t; }

}  // namespace pm_tile
