// Adjoint of the batched type-1 map on gfx950: a type-2 NUFFT (the +i sign of
// the series, eq. series) followed by the chain rule through the per-point
// strength c_j = w_j W(x_j) h_j.
//
// For a cotangent g on the coefficients, u_j = scale Re sum_k g_k exp(+i k.x_j)
// and its coordinate derivatives come from three fine grids: the pre-corrected
// spectrum (g_k divided by the kernel factors p(kx) p(ky), the inverse of
// Step 4) made Hermitian, and the same times i kx and i ky, each brought to the
// grid by an inverse FFT; the points then gather W x W taps from each grid with
// the same spreading kernel.  The three grids of a whole cell do not fit in
// LDS: one launch transforms the columns of every cell (adj_cols_kernel), then
// each work item of the next builds one row band of the grids (plus the
// kernel's halo) from them and serves the points whose footprint starts in
// that band.  Nothing of the forward pass is stored.
#include <algorithm>
#include <string>

#include "device_common.h"
#include "launch.h"
#include "plan.h"

namespace enufft {

// Elements of the staging area: the cell's N1 N2 complex coefficients, the
// K1 + 1 and K2 + 1 deconvolution factors, then N1 N2 keep bytes.
__host__ __device__ inline size_t adj_stage_elems(const Geom &g, size_t elem) {
  const size_t M = (size_t)g.N1 * g.N2;
  return 2 * M + (g.K1 + 1) + (g.K2 + 1) + (M + elem - 1) / elem;
}

// Copy the cell's cotangent spectrum, its keep bytes and the deconvolution
// factors into the staging area.  Every thread issues all of its global loads
// before it stores any (the loads are unconditional, clamped to the last
// element), so the copy costs about one memory latency instead of one per
// element.
template <typename T, int NT>
__device__ __forceinline__ void stage_spectrum(const AdjArgs<T> &a, const T *gc, int cell, T *st) {
  const Geom &g = a.g;
  const int M = g.N1 * g.N2, n = 2 * M;
  constexpr int U = 16;
  for (int base = 0; base < n; base += U * NT) {
    T v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = gc[min(base + u * NT + (int)threadIdx.x, n - 1)];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = base + u * NT + threadIdx.x;
      if (i < n) st[i] = v[u];
    }
  }
  T *sdx = st + n, *sdy = sdx + g.K1 + 1;
  for (int i = threadIdx.x; i <= g.K1; i += NT) sdx[i] = a.decon_x[i];
  for (int i = threadIdx.x; i <= g.K2; i += NT) sdy[i] = a.decon_y[i];
  if (a.keep) {
    const uint8_t *kp = a.keep + (int64_t)cell * M;
    uint8_t *sk = reinterpret_cast<uint8_t *>(sdy + g.K2 + 1);
    for (int base = 0; base < M; base += U * NT) {
      uint8_t v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) v[u] = kp[min(base + u * NT + (int)threadIdx.x, M - 1)];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int i = base + u * NT + threadIdx.x;
        if (i < M) sk[i] = v[u];
      }
    }
  }
  __syncthreads();
}

// First-step accessor of the column transforms: load(i) forms bin i (fine
// row, natural order) of column kx of the Hermitian, pre-corrected spectrum
// from the staged copy: (G(kx, ky) + conj G(-kx, -ky)) / 2 divided by the
// kernel transform, each term zero outside the mode box, with the
// retained-power factor two_lam on kept modes (1 without a keep mask); with
// yderiv, times i ky.  store() writes the column workspace.
template <typename T>
struct ColSpecAcc {
  const T *sf, *sdx, *sdy;
  const uint8_t *kp;
  T two_lam;
  T *col;   // column kx of the workspace (interleaved complex, row pitch cpitch)
  int cpitch, kx, n2, K2, N1, lo1, lo2, hi1, hi2;
  bool yderiv;
  __device__ void load(int bin, T &re, T &im) const {
    const int ky = bin <= n2 / 2 ? bin : bin - n2;   // signed frequency of this bin
    T hr = 0, hi = 0;
    if (ky >= -K2 && ky <= K2) {
      const T s = sdx[kx] * sdy[ky < 0 ? -ky : ky];
      if (kx <= hi1 && ky >= lo2 && ky <= hi2) {
        const int m = (ky - lo2) * N1 + (kx - lo1);
        const T sc = kp ? (kp[m] ? two_lam : T(0)) : T(1);
        hr += sc * sf[2 * m];
        hi += sc * sf[2 * m + 1];
      }
      if (-kx >= lo1 && -ky >= lo2 && -ky <= hi2) {
        const int m = (-ky - lo2) * N1 + (-kx - lo1);
        const T sc = kp ? (kp[m] ? two_lam : T(0)) : T(1);
        hr += sc * sf[2 * m];
        hi -= sc * sf[2 * m + 1];
      }
      hr *= T(0.5) * s;
      hi *= T(0.5) * s;
      if (yderiv) {
        const T t = hr;
        hr = -T(ky) * hi;
        hi = T(ky) * t;
      }
    }
    re = hr;
    im = hi;
  }
  __device__ void store(int i, T re, T im) const {
    col[i * cpitch] = re;
    col[i * cpitch + 1] = im;
  }
};

// Second step of the column transforms, out of place: item k1 of column kx
// computes fine rows y = k1 + A k2 and writes those of the band (band row r
// holds fine row (y0 + r) mod n2, r < rows) to the band spectra db
// ([row][kx] complex).
template <int A, int B, typename T>
__device__ __forceinline__ void col_step2_band(const T *col, int cpitch, int k1, int n2, T *db, int per, int kx,
                                               int rows, int y0) {
  T re[B], im[B];
#pragma unroll
  for (int b = 0; b < B; ++b) {
    re[b] = col[(k1 * B + b) * cpitch];
    im[b] = col[(k1 * B + b) * cpitch + 1];
  }
  dft_reg<B, true, T>(re, im);
#pragma unroll
  for (int k2 = 0; k2 < B; ++k2) {
    // band row r, and r + n2 too when the band's halo wraps onto its own
    // first rows (one band per cell: rows = n2 + W)
    const int r = (k1 + A * k2 - y0) & (n2 - 1);
    if (r < rows) {
      db[2 * (r * per + kx)] = re[k2];
      db[2 * (r * per + kx) + 1] = im[k2];
    }
    if (r + n2 < rows) {
      db[2 * ((r + n2) * per + kx)] = re[k2];
      db[2 * ((r + n2) * per + kx) + 1] = im[k2];
    }
  }
}

// One column pass: the inverse transforms along y of columns kx = 0..K1 of the
// spectrum (times i ky with yderiv), formed from the staged copy in the first
// step and written to the band spectra db by the second.
template <typename T, int NT>
__device__ __forceinline__ void column_pass(const AdjArgs<T> &a, const T *st, const T *tw2, T two_lam, T *ws, int cpitch,
                            bool yderiv, T *db, int rows, int y0) {
  const Geom &g = a.g;
  const int per = g.K1 + 1, n2 = g.n2, M = g.N1 * g.N2;
  const int A = fft_A(n2), B = fft_B(n2);
  ColSpecAcc<T> acc;
  acc.sf = st;
  acc.sdx = st + 2 * M;
  acc.sdy = acc.sdx + per;
  acc.kp = a.keep ? reinterpret_cast<const uint8_t *>(acc.sdy + g.K2 + 1) : nullptr;
  acc.two_lam = two_lam;
  acc.cpitch = cpitch;
  acc.n2 = n2; acc.K2 = g.K2; acc.N1 = g.N1; acc.lo1 = g.lo1; acc.lo2 = g.lo2;
  acc.hi1 = g.lo1 + g.N1 - 1; acc.hi2 = g.lo2 + g.N2 - 1;
  acc.yderiv = yderiv;
  // Consecutive lanes take consecutive columns (the column is the fast index of
  // both steps), so their LDS words are adjacent: the staged coefficients of
  // consecutive kx, the workspace elements 2 kx apart, the band spectra of
  // consecutive kx.  (With the transform position as the fast index, lanes
  // were a row of the staged box, or 8 or 16 workspace rows, apart: 8- and
  // 16-way bank conflicts.)
  for (int it = threadIdx.x; it < per * B; it += NT) {
    const int b = it / per, q = it - b * per;
    ColSpecAcc<T> c = acc;
    c.kx = q;
    c.col = ws + 2 * q;
    fft4_dispatch<true, 1, T>(n2, c, b, tw2);
  }
  __syncthreads();
  for (int it = threadIdx.x; it < per * A; it += NT) {
    const int k1 = it / per, q = it - k1 * per;
    const T *col = ws + 2 * q;
    switch (n2) {
      case 16: col_step2_band<4, 4, T>(col, cpitch, k1, n2, db, per, q, rows, y0); break;
      case 32: col_step2_band<8, 4, T>(col, cpitch, k1, n2, db, per, q, rows, y0); break;
      case 64: col_step2_band<8, 8, T>(col, cpitch, k1, n2, db, per, q, rows, y0); break;
      default: col_step2_band<16, 8, T>(col, cpitch, k1, n2, db, per, q, rows, y0); break;
    }
  }
  __syncthreads();
}

// Second step of the row transforms, writing natural column order.  Item k1
// of a row computes bins k1 + A k2 (k2 = 0 .. B - 1) from positions k1 B + b
// and stores bin k at column k, and again at n1 + k for k < W - 1 (the first
// W - 1 columns repeated after the last, so a footprint's W taps in a row are
// W consecutive elements).  The store lands on positions other items of the
// same row still read, so the A items of a row must be one wave's lanes: a
// wave's LDS accesses complete in issue order and every item loads before it
// stores.  With A | 64 and 64 | NT, the items q A .. q A + A - 1 of the
// batched loop below always share a wave.  The first step stores with
// fft4_step1_swz (the inputs of item k1 sit at k1 B + (b ^ fft_swz(k1, B))).
template <int A, int B, typename T, typename Acc>
__device__ __forceinline__ void row_step2_natural(const Acc &acc, int k1, int n, int wrap) {
  T re[B], im[B];
  const int sw = fft_swz(k1, B);
#pragma unroll
  for (int b = 0; b < B; ++b) acc.load(k1 * B + (b ^ sw), re[b], im[b]);
  dft_reg<B, true, T>(re, im);
#pragma unroll
  for (int k2 = 0; k2 < B; ++k2) {
    const int k = k1 + A * k2;
    acc.store(k, re[k2], im[k2]);
    if (k < wrap) acc.store(n + k, re[k2], im[k2]);
  }
}

// The batched inverse row transforms: step 1 through make1(q) (forming the
// spectra), step 2 in place through make2(q) into natural column order.
template <int NT, typename T, typename Make1, typename Make2>
__device__ __forceinline__ void row_ifft_natural(int n, int count, const T *tw, int wrap, const Make1 &make1,
                                                 const Make2 &make2) {
  static_assert(NT % 64 == 0, "whole waves");
  const int A = fft_A(n), B = fft_B(n), la = fft_logA(n), lb = fft_logB(n);
  for (int it = threadIdx.x; it < count * B; it += NT) {
    const int q = it >> lb, b = it & (B - 1);
    fft4_step1_swz_dispatch<true, T>(n, make1(q), b, tw);
  }
  __syncthreads();
  for (int it = threadIdx.x; it < count * A; it += NT) {
    const int q = it >> la, k1 = it & (A - 1);
    switch (n) {
      case 16: row_step2_natural<4, 4, T>(make2(q), k1, n, wrap); break;
      case 32: row_step2_natural<8, 4, T>(make2(q), k1, n, wrap); break;
      case 64: row_step2_natural<8, 8, T>(make2(q), k1, n, wrap); break;
      default: row_step2_natural<16, 8, T>(make2(q), k1, n, wrap); break;
    }
  }
  __syncthreads();
}

// First-step accessor of the row transforms: load(k) forms bin k of the row's
// spectrum from column data db ([row][kx] complex, kx = 0..K1): for a (u, du/dx)
// row, (1 - k) D(k); for a pair of rows (row, row + 1), D_row(k) + i D_row+1(k);
// D(-k) = conj D(k), zero beyond K1.  store() writes the grid row like
// StridedPairAcc.  The loads are unconditional (bins beyond K1 read bin K1), so
// those of one transform are in flight together when db is global memory.
template <typename T>
struct RowSpecAcc {
  const T *db;
  T *r0, *r1;
  int stride, row, per, n1, K1;
  bool pair;
  __device__ void load(int k, T &re, T &im) const {
    using V2 = typename vec2<T>::type;
    const int kk = k <= n1 / 2 ? k : n1 - k;
    const bool neg = k != kk, in = kk <= K1;
    const V2 *d = reinterpret_cast<const V2 *>(db) + (row * per + (in ? kk : K1));
    const V2 v = d[0];
    const T di = neg ? -v.y : v.y;
    if (!pair) {
      const T kf = neg ? -T(kk) : T(kk);
      re = in ? v.x - kf * v.x : T(0);
      im = in ? di - kf * di : T(0);
    } else {
      const V2 w = d[per];
      const T bi = neg ? -w.y : w.y;
      re = in ? v.x - bi : T(0);
      im = in ? di + w.x : T(0);
    }
  }
  __device__ void store(int i, T re, T im) const {
    r0[i * stride] = re;
    r1[i * stride] = im;
  }
};

// ------------------------------------------------------------------ banded adjoint

// First-step accessor of the column transforms from global memory: as
// ColSpecAcc, reading the cell's coefficients, keep bytes and deconvolution
// factors in place.  A bin's loads are issued together (without a keep mask the
// coefficients' bytes are read in its place, so no test of its presence parts them); with
// that test between them a bin cost three latencies and 4,000 cells of FP32 columns
// 325 us.  (All bins' loads at once, with factors for the masks, need 184 registers in
// FP32 and 266 in FP64: 2 us less for 60 cells, 100 more for 4,000.)
template <typename T>
struct ColSpecGlobal {
  const typename vec2<T>::type *sf;
  const T *dx, *dy;
  const uint8_t *kp;
  T two_lam, dropped;   // factors of kept and of other modes (both 1 without a mask)
  T *col;
  int cpitch, kx, n2, K2, N1, lo1, lo2, hi1, hi2;
  bool yderiv;
  __device__ void load(int bin, T &re, T &im) const {
    const int ky = bin <= n2 / 2 ? bin : bin - n2;
    const bool in = ky >= -K2 && ky <= K2;
    const bool p = in && kx <= hi1 && ky >= lo2 && ky <= hi2;
    const bool q = in && -kx >= lo1 && -ky >= lo2 && -ky <= hi2;
    const int mp = p ? (ky - lo2) * N1 + (kx - lo1) : 0, mq = q ? (-ky - lo2) * N1 + (-kx - lo1) : 0;
    const auto vp = sf[mp], vq = sf[mq];
    const T sp = kp[mp] ? two_lam : dropped, sq = kp[mq] ? two_lam : dropped;
    const T s = T(0.5) * (dx[kx] * dy[in ? (ky < 0 ? -ky : ky) : 0]);
    T hr = p ? sp * vp.x : T(0), hi = p ? sp * vp.y : T(0);
    hr += q ? sq * vq.x : T(0);
    hi -= q ? sq * vq.y : T(0);
    hr *= s;
    hi *= s;
    re = !in ? T(0) : yderiv ? -T(ky) * hi : hr;
    im = !in ? T(0) : yderiv ? T(ky) * hr : hi;
  }
  __device__ void store(int i, T re, T im) const {
    col[i * cpitch] = re;
    col[i * cpitch + 1] = im;
  }
};

constexpr int ADJ_COLS_THREADS = 192;
constexpr int ADJ_COLS_GROUP = 12;   // columns of one workgroup, at most

__host__ __device__ inline int adj_col_groups(const Geom &g) {
  return (g.K1 + 1 + ADJ_COLS_GROUP - 1) / ADJ_COLS_GROUP;
}

// Column spectra of the cells cell0 .. : a.cols holds, per cell, `nset` blocks
// [n2][K1 + 1] complex, the inverse transforms along y of the pre-corrected
// spectrum (set 0) and of i ky times it (set 1).  One workgroup per (cell, set,
// group of up to 12 columns): the columns are independent, so a call with few
// cells still fills many CUs.  They are transformed once per cell here: inside the
// band kernel every band (32 of four rows each in FP64 at 64 x 64 modes and W = 12,
// whose column workspace left no room for more) and every chunk of a cell had
// repeated both column passes.  64 hexagons of 2.07e6 unordered samples in all, FP64,
// 64 x 64 modes, W = 12: this launch 16 us, the bands' 324 us (four bands of 32
// rows); the one launch before took 10.0 ms, with the exact kernel (a square root, a
// division and an exponential per tap) and one lane in 32 gathering.
template <typename T>
__global__ __launch_bounds__(ADJ_COLS_THREADS) void adj_cols_kernel(AdjArgs<T> a, int nset) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  constexpr int NT = ADJ_COLS_THREADS;
  const Geom &g = a.g;
  const int per = g.K1 + 1, ngrp = adj_col_groups(g), cg = (per + ngrp - 1) / ngrp;
  const int n2 = g.n2, A = fft_A(n2), B = fft_B(n2);
  int b = blockIdx.x;
  const int grp = b % ngrp;
  b /= ngrp;
  const int set = b % nset, lc = b / nset, cell = a.cell0 + lc;
  const int c0 = grp * cg, nc = min(cg, per - c0);
  if (nc <= 0) return;
  T *tw2 = reinterpret_cast<T *>(smem_raw), *ws = tw2 + 2 * n2;
  for (int i = threadIdx.x; i < 2 * n2; i += NT) tw2[i] = a.tw2[i];
  __syncthreads();
  ColSpecGlobal<T> acc;
  acc.sf = reinterpret_cast<const typename vec2<T>::type *>(a.fbar) + (int64_t)cell * g.N1 * g.N2;
  acc.dx = a.decon_x;
  acc.dy = a.decon_y;
  acc.kp = a.keep ? a.keep + (int64_t)cell * g.N1 * g.N2 : reinterpret_cast<const uint8_t *>(acc.sf);
  // the reconstruction's coefficients are kept or dropped, not weighted
  acc.two_lam = a.rec_part || !a.keep ? T(1) : T(2.0 * (a.lam ? a.lam[cell] : 1.0));
  acc.dropped = a.keep ? T(0) : T(1);
  acc.cpitch = 2 * cg + 2;
  acc.n2 = n2; acc.K2 = g.K2; acc.N1 = g.N1; acc.lo1 = g.lo1; acc.lo2 = g.lo2;
  acc.hi1 = g.lo1 + g.N1 - 1; acc.hi2 = g.lo2 + g.N2 - 1;
  acc.yderiv = set == 1;
  for (int it = threadIdx.x; it < nc * B; it += NT) {
    const int bb = it / nc, q = it - bb * nc;
    ColSpecGlobal<T> c = acc;
    c.kx = c0 + q;
    c.col = ws + 2 * q;
    fft4_dispatch<true, 1, T>(n2, c, bb, tw2);
  }
  __syncthreads();
  T *db = a.cols + ((int64_t)lc * nset + set) * n2 * per * 2;
  for (int it = threadIdx.x; it < nc * A; it += NT) {
    const int k1 = it / nc, q = it - k1 * nc;
    const T *col = ws + 2 * q;
    switch (n2) {
      case 16: col_step2_band<4, 4, T>(col, acc.cpitch, k1, n2, db, per, c0 + q, n2, 0); break;
      case 32: col_step2_band<8, 4, T>(col, acc.cpitch, k1, n2, db, per, c0 + q, n2, 0); break;
      case 64: col_step2_band<8, 8, T>(col, acc.cpitch, k1, n2, db, per, c0 + q, n2, 0); break;
      default: col_step2_band<16, 8, T>(col, acc.cpitch, k1, n2, db, per, c0 + q, n2, 0); break;
    }
  }
}

constexpr int ADJ_QCAP = 128;   // per-wave queue of the band's points (entries)

// LDS of a band item: the grid planes (three for the gradients: rows of
// interleaved (u, du/dx) and rows of du/dy; one, of u, for the FP64 reconstruction),
// the row twiddles and the per-wave queues of the band's points.
struct BandLayout {
  int rows;       // band rows including halo = band_rows + W, even
  int apitch;     // grid row pitch (elements) = n1 + W - 1, rounded up to even: the first W - 1
                  // columns are repeated after the last, so a footprint's W columns are contiguous
  size_t gy_off, tw_off;   // element offsets
  size_t q_off, total;     // bytes
};

__host__ __device__ inline BandLayout band_layout(const Geom &g, int W, int band_rows, size_t elem, bool recon,
                                                  int threads) {
  BandLayout L;
  L.rows = band_rows + W;
  L.apitch = (g.n1 + W - 1 + 1) & ~1;
  const size_t gsz = (size_t)L.rows * L.apitch;
  L.gy_off = 2 * gsz;
  L.tw_off = (recon ? 1 : 3) * gsz;
  L.q_off = (L.tw_off + 2 * (size_t)g.n1) * elem;
  // a band that is the whole grid serves every point and queues none
  L.total = L.q_off + (band_rows < g.n2 ? (size_t)(threads / 64) * ADJ_QCAP * sizeof(int) : 0);
  return L;
}

// What a point's interpolated u (and du/dx, du/dy) gives: the gradients, or in the
// reconstruction mode the error sums.
template <typename T, bool RECON>
__device__ __forceinline__ void finish_point(const AdjArgs<T> &a, int64_t j, T xj, T yj, T hj, T wj, T cx, T cy, T R, T pr,
                                             T u, T ux, T uy, double (&acc)[3]) {
  if constexpr (RECON) {
    const double t = (double)(hj * hann_w(a.window_kind, xj, yj, cx, cy, R, pr));
    const double d = t - (double)u;
    acc[0] += d * d;
    acc[1] += t * t;
    acc[2] += (double)wj * t * t;
    if (a.grad_h) a.grad_h[j] = u;
    return;
  }
  T dWx, dWy;
  const T Wv = hann_wg(a.window_kind, xj, yj, cx, cy, R, pr, dWx, dWy);
  if (a.grad_h) a.grad_h[j] = wj * Wv * u;
  if (a.grad_x || a.grad_y) {
    const T wh = wj * hj;
    if (a.grad_x) a.grad_x[j] = wh * (dWx * u + Wv * ux);
    if (a.grad_y) a.grad_y[j] = wh * (dWy * u + Wv * uy);
  }
}

// Gradients at one point whose footprint starts in band row r0, from the band's
// three grids (W x W taps each); the chain rule through the strength
// c_j = w_j W(x_j) h_j turns the interpolated u, du/dx, du/dy into dL/dh,
// dL/dx, dL/dy.
//
// RECON: the reconstruction mode.  Only u is interpolated; it is the truncated
// series h_rec(x_j) (the plan's scale is not applied in this mode), stored to
// grad_h when given, and the point adds (t - h_rec)^2, t^2 and w t^2 to acc, with
// t = W(x_j) h_j the windowed height.
//
// POLY: the taps are the plan's polynomials (FP32 up to W = 8, FP64), taken in
// mirror pairs; otherwise psi itself.  Either is fixed at compile time (a
// run-time choice makes the compiler keep the taps in scratch).
template <typename T, int W, bool POLY, bool RECON>
__device__ __forceinline__ void gather_point(const AdjArgs<T> &a, const T *G, const T *Gy, int apitch, int r0,
                                             const FineCoord<T> &fy, int64_t j, T xj, T yj, T hj, T wj, T cx, T cy,
                                             T R, T pr, double (&acc)[3]) {
  const Geom &g = a.g;
  const T halfw = T(W) / T(2);
  const FineCoord<T> fx = fine_coord<T>(xj, a.s1_hi, a.s1_lo, halfw);
  T kx[W];
  T u = 0, ux = 0, uy = 0;
  using V2 = typename vec2<T>::type;
  // rows in natural column order with the wrap-around columns repeated: the
  // W taps of a row are W consecutive elements from one base address
  const int e0 = r0 * apitch + (fx.i0 & (g.n1 - 1));
  const V2 *puv = reinterpret_cast<const V2 *>(G) + e0;
  const T *p1 = (RECON ? G : Gy) + e0;
  auto row = [&](int dy, T kyv) {
    T su = 0, sx = 0, sy = 0;
    const V2 *q = puv + dy * apitch;
    const T *qy = p1 + dy * apitch;
#pragma unroll
    for (int dx = 0; dx < W; ++dx) {
      if constexpr (RECON) {
        su += kx[dx] * qy[dx];
      } else {
        const V2 v = q[dx];
        su += kx[dx] * v.x;
        sx += kx[dx] * v.y;
        sy += kx[dx] * qy[dx];
      }
    }
    u += kyv * su;
    if constexpr (!RECON) {
      ux += kyv * sx;
      uy += kyv * sy;
    }
  };
  if constexpr (POLY && sizeof(T) == 8) {
    es_taps64<W>(tap_u64(fx, double(W) * 0.5), a.es64, kx);
    const double uyv = tap_u64(fy, double(W) * 0.5), sy2 = uyv * uyv;
    // two rows at a time, so the loads of all W rows are not held in registers together
    double ta, tb;
    tap_pair64<W>(a.es64, 0, uyv, sy2, ta, tb);
    row(0, ta);
    row(W - 1, tb);
#pragma unroll 1
    for (int d = 1; d < W / 2; ++d) {
      poly64_pair_eval(poly64_pair(a.es64, d), uyv, sy2, ta, tb);
      row(d, ta);
      row(W - 1 - d, tb);
    }
  } else if constexpr (POLY) {
    T ky[W];
    es_taps_poly<W>(fx, float(W) * 0.5f, a.es, kx);
    es_taps_poly<W>(fy, float(W) * 0.5f, a.es, ky);
#pragma unroll
    for (int dy = 0; dy < W; ++dy) row(dy, ky[dy]);
  } else {
    const T zsc = T(2) / T(W);
#pragma unroll
    for (int d = 0; d < W; ++d) kx[d] = ker_eval(fx.offset(d) * zsc, a.beta);
    // one row at a time, so the loads of all W rows are not hoisted together
#pragma unroll 1
    for (int dy = 0; dy < W; ++dy) row(dy, ker_eval(fy.offset(dy) * zsc, a.beta));
  }
  finish_point<T, RECON>(a, j, xj, yj, hj, wj, cx, cy, R, pr, u, ux, uy, acc);
}

// FP64 with the kernel polynomial, W > 8: the points of a wave's lanes, four at a time,
// one per row of sixteen lanes.  Lane d of a row evaluates tap d of its point along both
// axes and sums its column down the W rows (the y taps broadcast along the row), so an
// instruction reads W consecutive cells per point; one point per lane read 64 unrelated
// ones, two thirds of whose LDS cycles were bank conflicts.  The column sums times
// their x taps are then added up within the row.  64 cells of 2.1e6 points at W = 12: 324
// to 304 us (60 cycles per point of a CU, its arithmetic and its LDS reads half each;
// 13 % are the bands' row transforms and a quarter the uneven bands of 2.5 items per CU).
//
// The row sums of four points are merged as they are halved: after two steps each
// quarter of a row holds one point's, at the cost of 1.7 plain reductions instead of 4.
template <int N>
__device__ __forceinline__ double row_ror(double v) {   // lane i takes lane (i - N) mod 16 of its row
  return __hiloint2double(__builtin_amdgcn_mov_dpp(__double2hiint(v), 0x120 + N, 0xf, 0xf, true),
                          __builtin_amdgcn_mov_dpp(__double2loint(v), 0x120 + N, 0xf, 0xf, true));
}
template <int X>
__device__ __forceinline__ double quad_xor(double v) {   // lane i takes lane i ^ X of its quad
  constexpr int P = X == 1 ? 0xb1 : 0x4e;                // quad_perm [1,0,3,2] or [2,3,0,1]
  return __hiloint2double(__builtin_amdgcn_mov_dpp(__double2hiint(v), P, 0xf, 0xf, true),
                          __builtin_amdgcn_mov_dpp(__double2loint(v), P, 0xf, 0xf, true));
}
// The rows of a lane's column, the y tap of row R from lane R of its row.
template <int W, bool RECON, int R = 0>
__device__ __forceinline__ void column_rows(const double2 *q, const double *qy, int apitch, double ky, double (&s)[3]) {
  if constexpr (R < W) {
    const double k = row_bcast<R>(ky);
    if constexpr (RECON) {
      s[0] = fma(k, *qy, s[0]);
    } else {
      const double2 v = *q;
      s[0] = fma(k, v.x, s[0]);
      s[1] = fma(k, v.y, s[1]);
      s[2] = fma(k, *qy, s[2]);
    }
    column_rows<W, RECON, R + 1>(q + apitch, qy + apitch, apitch, ky, s);
  }
}
// Quarters of a row afterwards: the sums of v[0], v[2], v[1], v[3], in all their lanes.
__device__ __forceinline__ double row_sums4(const double (&v)[4], int li) {
  const bool up = li & 8, odd = li & 4;
  const double t0 = (up ? v[1] : v[0]) + row_ror<8>(up ? v[0] : v[1]);
  const double t1 = (up ? v[3] : v[2]) + row_ror<8>(up ? v[2] : v[3]);
  const double send = odd ? t0 : t1;
  const double below = row_ror<4>(send), above = row_ror<12>(send);   // both in every lane
  double r = (odd ? t1 : t0) + (odd ? below : above);
  r += quad_xor<1>(r);
  r += quad_xor<2>(r);
  return r;
}
template <int W, bool RECON, int L = 0>
__device__ __forceinline__ void row_points(const double *G, const double *Gy, int apitch, const RowTap<W> &tap, int li,
                                           double ux, double uy, int o, double (&su)[4], double (&sx)[4],
                                           double (&sy)[4]) {
  if constexpr (L < 4) {
    const int op = row_bcast<L>(o);
    const double vx = row_bcast<L>(ux), vy = row_bcast<L>(uy);
    su[L] = sx[L] = sy[L] = 0.0;
    if (op >= 0 && li < W) {
      const double kx = tap(vx), ky = tap(vy);
      double s[3] = {0.0, 0.0, 0.0};
      column_rows<W, RECON>(reinterpret_cast<const double2 *>(G) + op + li, (RECON ? G : Gy) + op + li, apitch, ky, s);
      su[L] = kx * s[0];
      if constexpr (!RECON) {
        sx[L] = kx * s[1];
        sy[L] = kx * s[2];
      }
    }
    row_points<W, RECON, L + 1>(G, Gy, apitch, tap, li, ux, uy, o, su, sx, sy);
  }
}
// e: the first element of the lane's own point, -1 for none.  The lane's u, ux, uy.
template <int W, bool RECON>
__device__ __forceinline__ void gather_rows(const double *G, const double *Gy, int apitch, const RowTap<W> &tap, double ux,
                                            double uy, int e, double &u, double &gx, double &gy) {
  const int lane = threadIdx.x & 63, li = lane & 15;
  double ru = 0.0, rx = 0.0, ry = 0.0;
#pragma unroll 1
  for (int q = 0; q < 4; ++q) {
    double su[4], sx[4], sy[4];
    row_points<W, RECON>(G, Gy, apitch, tap, li, ux, uy, e, su, sx, sy);
    const double tu = row_sums4(su, li);
    const bool mine = (li & 3) == q;   // lane 4 k + q of a row keeps quarter k's sums of round q
    ru = mine ? tu : ru;
    if constexpr (!RECON) {
      const double tx = row_sums4(sx, li), ty = row_sums4(sy, li);
      rx = mine ? tx : rx;
      ry = mine ? ty : ry;
    }
    ux = row_next4(ux); uy = row_next4(uy); e = row_next4(e);
  }
  // the point of lane 4 q + L: quarter L (1 and 2 exchanged), its lane q
  const int L = li & 3, src = (lane & 48) + 4 * (L == 1 ? 2 : L == 2 ? 1 : L) + (li >> 2);
  u = __shfl(ru, src, 64);
  if constexpr (!RECON) {
    gx = __shfl(rx, src, 64);
    gy = __shfl(ry, src, 64);
  }
}

// All points of one item.  When the band is the whole grid every point is
// served: wave w takes blocks of 64 consecutive points, one per lane, each lane's
// next point loaded while the current one is gathered.  Otherwise every y of the
// item is read and the points of the band are queued per wave and gathered 64 at
// a time: served where they stand, only one lane in `bands` would be active for
// points in no spatial order, at the cost of a whole wave's gather each time.  Up to
// W = 8 a wave whose points all lie in the band serves them where they stand, as raster
// points mostly do.  The waves take the item's blocks of 64 points in turn: with blocks of
// 256 to a wave an item of 600 points had kept three of the eight waves busy.  Both
// together, FP32, W = 8, raster points: 4,000 cells of 600 1,010 to 927 us, 60 of 28,000
// 106.5 to 103.3; FP64, W = 10, 1,500 cells of 600 936 to 620 us, of which the column
// launch's loads (ColSpecGlobal) are part.
template <typename T, int W, int NT, bool POLY, bool RECON>
__device__ __forceinline__ void gather_item(const AdjArgs<T> &a, const T *G, const T *Gy, int apitch, int *queue,
                                            int band_lo, int64_t begin, int64_t end, T cx, T cy, T R,
                                            double (&acc)[3]) {
  const T pr = R > T(0) ? T(M_PI) / R : T(0);
  const T halfw = T(W) / T(2);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int mask2 = a.g.n2 - 1;
  if (begin >= end) return;
  constexpr bool kRows = POLY && sizeof(T) == 8 && W > 8;
  typename std::conditional<kRows, RowTap<W>, int>::type tap;
  if constexpr (kRows) tap.init(a.es64, lane & 15);
  // the whole wave: point j per lane (on: a point at all), its footprint from row r0 of G
  auto rows = [&](bool on, int64_t j, T xj, T yj, T hj, T wj, int lo) {
    if constexpr (kRows) {
      const FineCoord<T> fx = fine_coord<T>(xj, a.s1_hi, a.s1_lo, halfw), fy = fine_coord<T>(yj, a.s2_hi, a.s2_lo, halfw);
      const int e = on ? ((fy.i0 & mask2) - lo) * apitch + (fx.i0 & (a.g.n1 - 1)) : -1;
      T u = 0, ux = 0, uy = 0;
      gather_rows<W, RECON>(G, Gy, apitch, tap, tap_u64(fx, halfw), tap_u64(fy, halfw), e, u, ux, uy);
      if (on) finish_point<T, RECON>(a, j, xj, yj, hj, wj, cx, cy, R, pr, u, ux, uy, acc);
    }
  };
  if (a.band_rows > mask2) {
    struct Pt {
      T x, y, h, w;
    };
    auto load = [&](Pt &b, int64_t i) {
      const int64_t ic = i < end ? i : end - 1;   // past the end: re-read the last point (unused)
      b.x = a.x[ic]; b.y = a.y[ic]; b.h = a.h[ic]; b.w = a.w[ic];
    };
    auto step = [&](const Pt &b, int64_t i) {
      if constexpr (kRows) {
        rows(i < end, i, b.x, b.y, b.h, b.w, 0);
      } else if (i < end) {
        const FineCoord<T> fy = fine_coord<T>(b.y, a.s2_hi, a.s2_lo, halfw);
        gather_point<T, W, POLY, RECON>(a, G, Gy, apitch, fy.i0 & mask2, fy, i, b.x, b.y, b.h, b.w, cx, cy, R, pr,
                                        acc);
      }
    };
    constexpr int64_t stride = NT;
    int64_t i = begin + threadIdx.x;
    Pt b0, b1;
    load(b0, i);
    for (; i - lane < end; i += 2 * stride) {
      load(b1, i + stride);
      step(b0, i);
      load(b0, i + 2 * stride);
      step(b1, i + stride);
    }
    return;
  }
  constexpr int U = 4;
  int *wq = queue + wave * ADJ_QCAP;
  // the queue's entry of a lane (rows of lanes: neighbours of the queue in different rows,
  // so a short one fills all)
  const int slot = kRows ? (lane & 15) * 4 + (lane >> 4) : lane;
  auto serve = [&](bool on, int64_t j) {
    if constexpr (kRows) {
      rows(on, j, a.x[j], a.y[j], a.h[j], a.w[j], band_lo);
    } else if (on) {
      const T xj = a.x[j], yj = a.y[j], hj = a.h[j], wj = a.w[j];
      const FineCoord<T> fy = fine_coord<T>(yj, a.s2_hi, a.s2_lo, halfw);
      gather_point<T, W, POLY, RECON>(a, G, Gy, apitch, (fy.i0 & mask2) - band_lo, fy, j, xj, yj, hj, wj, cx, cy, R,
                                      pr, acc);
    }
  };
  auto order = [] {   // a wave's LDS accesses complete in issue order; keep the compiler to it
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  int nq = 0;   // queued points (the same in every lane)
  T yb[U];
  auto load = [&](int64_t p) {
#pragma unroll
    for (int u = 0; u < U; ++u) yb[u] = a.y[min(p + u * NT + (int)threadIdx.x, end - 1)];
  };
  load(begin);
  for (int64_t p = begin; p < end; p += U * NT) {
    bool in[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int r0 = (fine_coord<T>(yb[u], a.s2_hi, a.s2_lo, halfw).i0 & mask2) - band_lo;
      in[u] = p + u * NT + (int)threadIdx.x < end && r0 >= 0 && r0 < a.band_rows;
    }
    load(p + U * NT);
#pragma unroll 1
    for (int u = 0; u < U; ++u) {
      const bool on = u == 0 ? in[0] : u == 1 ? in[1] : u == 2 ? in[2] : in[3];
      const uint64_t m = __ballot(on);
      if (m == 0) continue;
      int64_t j = p + u * NT + (int)threadIdx.x;
      if (kRows || m != ~0ull) {
        if (on) {
          const int pos = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
          wq[nq + pos] = (int)(j - begin);   // nq < 64 here, so nq + pos < ADJ_QCAP
        }
        nq += __popcll(m);
        if (nq < 64) continue;
        order();
        nq -= 64;
        j = begin + wq[slot];
        const int rest = lane < nq ? wq[64 + lane] : 0;
        order();
        if (lane < nq) wq[lane] = rest;
        order();
      }
      serve(true, j);
    }
  }
  order();
  if (nq > 0) serve(slot < nq, begin + wq[min(slot, nq - 1)]);
}

template <typename T, int W, int NT, bool POLY, bool RECON>
__global__ __launch_bounds__(NT) void adj_kernel(AdjArgs<T> a) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  T *sm = reinterpret_cast<T *>(smem_raw);
  __shared__ int s_item;
  const Geom &g = a.g;
  const BandLayout L = band_layout(g, W, a.band_rows, sizeof(T), RECON, NT);
  const int pitch = L.apitch;
  // gradients: rows of (u, du/dx) pairs (the real and imaginary parts of one
  // complex row transform, kept interleaved) in G, rows of du/dy in Gy;
  // reconstruction: rows of u in G
  T *G = sm, *Gy = sm + L.gy_off, *tw1 = sm + L.tw_off;
  int *queue = reinterpret_cast<int *>(smem_raw + L.q_off);
  const int per = g.K1 + 1, n1 = g.n1, n2 = g.n2, K1 = g.K1;
  // the transforms' twiddles stay in LDS for all items of this workgroup (the
  // barrier at the top of the item loop orders them before first use)
  for (int i = threadIdx.x; i < 2 * n1; i += NT) tw1[i] = a.tw1[i];
  for (;;) {
    if (threadIdx.x == 0) s_item = atomicAdd(a.work_counter, 1);
    __syncthreads();
    const int64_t idx = s_item;
    __syncthreads();
    if (idx >= a.n_items) break;
    const AdjItem it = a.items[idx];
    const int y0 = it.band * a.band_rows;   // fine row of band-local row 0
    const size_t set = (size_t)n2 * per * 2;
    const T *db0 = a.cols + (size_t)(it.cell - a.cell0) * (RECON ? 1 : 2) * set, *db1 = db0 + set;
    // Row stage, one batch of inverse transforms: the (u, du/dx) rows, spectrum
    // Z(k) = D(k) + i (i k D(k)) = (1 - k) D(k), stored interleaved in G, and
    // the du/dy row pairs, Z(k) = Dy_r(k) + i Dy_r+1(k), in Gy (RECON: row pairs of
    // u); the bins k < 0 are the conjugates of column -k.  The first step reads
    // the spectra from the cell's column data in global memory, the second writes
    // natural column order with the wrap-around columns; band rows = band_rows +
    // W and y0 are even, so the rows pair up exactly.
    const int nuv = RECON ? 0 : L.rows;
    row_ifft_natural<NT, T>(
        n1, nuv + L.rows / 2, tw1, W - 1,
        [&](int q) {
          RowSpecAcc<T> acc;
          const int r = q < nuv ? q : 2 * (q - nuv);
          acc.db = RECON || q < nuv ? db0 : db1;
          acc.row = (y0 + r) & (n2 - 1);
          acc.pair = q >= nuv;
          acc.per = per;
          acc.n1 = n1;
          acc.K1 = K1;
          acc.r0 = q < nuv ? G + 2 * r * pitch : (RECON ? G : Gy) + r * pitch;
          acc.r1 = q < nuv ? acc.r0 + 1 : acc.r0 + pitch;
          acc.stride = q < nuv ? 2 : 1;
          return acc;
        },
        [&](int q) {
          StridedPairAcc<T> acc;
          const int r = q < nuv ? q : 2 * (q - nuv);
          acc.r0 = q < nuv ? G + 2 * r * pitch : (RECON ? G : Gy) + r * pitch;
          acc.r1 = q < nuv ? acc.r0 + 1 : acc.r0 + pitch;
          acc.stride = q < nuv ? 2 : 1;
          return acc;
        });

    // Gather at the points of this band.
    const double *wn = a.windows + 3 * (int64_t)it.cell;
    double acc[3] = {0.0, 0.0, 0.0};
    gather_item<T, W, NT, POLY, RECON>(a, G, Gy, pitch, queue, y0, it.begin, it.end, T(wn[0]), T(wn[1]), T(wn[2]),
                                       acc);
    if constexpr (RECON) {
      // the item's three sums, reduced in a fixed order (waves, then lanes)
      __syncthreads();
      double *red = reinterpret_cast<double *>(sm);
      for (int k = 0; k < 3; ++k) {
        double v = acc[k];
        for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
        if ((threadIdx.x & 63) == 0) red[k * (NT / 64) + (threadIdx.x >> 6)] = v;
      }
      __syncthreads();
      if (threadIdx.x < 3) {
        double v = 0.0;
        for (int q = 0; q < NT / 64; ++q) v += red[threadIdx.x * (NT / 64) + q];
        a.rec_part[3 * idx + threadIdx.x] = v;
      }
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    __threadfence();
    const int old = atomicAdd(a.done_counter, 1);
    if (old == (int)gridDim.x - 1) {
      *a.work_counter = 0;
      *a.done_counter = 0;
    }
  }
}

constexpr int ADJ_THREADS = 512;

// Compiled with polynomial taps for FP32 (W <= ES_MAXW) and FP64, and with the exact
// kernel; the reconstruction in FP64 (FP32: rec_kernel below).
template <typename T, int W>
static const void *adj_fn(bool poly, bool recon) {
  if constexpr (sizeof(T) == 8) {
    if (recon)
      return poly ? (const void *)&adj_kernel<T, W, ADJ_THREADS, true, true>
                  : (const void *)&adj_kernel<T, W, ADJ_THREADS, false, true>;
  }
  if constexpr (sizeof(T) == 8 || W <= ES_MAXW) {
    if (poly) return (const void *)&adj_kernel<T, W, ADJ_THREADS, true, false>;
  }
  return recon ? nullptr : (const void *)&adj_kernel<T, W, ADJ_THREADS, false, false>;
}

template <typename T>
static const void *adj_fn_w(int W, bool poly, bool recon) {
  switch (W) {
    case 4: return adj_fn<T, 4>(poly, recon);
    case 6: return adj_fn<T, 6>(poly, recon);
    case 8: return adj_fn<T, 8>(poly, recon);
    case 10: return adj_fn<T, 10>(poly, recon);
    case 12: return adj_fn<T, 12>(poly, recon);
    case 14: return adj_fn<T, 14>(poly, recon);
    case 16: return adj_fn<T, 16>(poly, recon);
    default: return nullptr;
  }
}

// ------------------------------------------------------------------ FP32 reconstruction
//
// FP32 plans reconstruct from rows of (u, du/dx) like the gradients' (the du/dx half is
// transformed beside u and not read), in row bands that transform their own columns.  The
// pairing of rows that serves FP64 above would round u differently, by about 5e-8, which
// the per-cell FP64 sums of squared FP32 residuals follow; the same row transforms with
// only their real parts stored would need half the LDS and a single band at the 64 x 64
// box, and are not built.  (The arms for row pairs below are not taken; a build without
// them, and without the column pass's unused derivative, rounded u differently all the
// same, and moved the sums by 3e-8.)

struct RecLayout {
  int rows;       // band rows including halo = band_rows + W
  int apitch;     // grid row pitch (elements), as BandLayout
  int cpitch;     // column-workspace pitch (elements) = 2 (K1 + 1) + 2
  size_t db_off, ws_off, st_off;   // element offsets (the grid of (u, du/dx) pairs at 0)
  size_t tw_off;  // twiddles of the row (n1) and column (n2) transforms, interleaved complex
  size_t total;   // elements
};

__host__ __device__ inline RecLayout rec_layout(const Geom &g, int W, int band_rows, size_t elem) {
  RecLayout L;
  L.rows = band_rows + W;
  L.apitch = (g.n1 + W - 1 + 1) & ~1;
  L.cpitch = 2 * (g.K1 + 1) + 2;
  const size_t gsz = 2 * (size_t)L.rows * L.apitch;
  // the column workspace and the staging area behind it alias the grid (they
  // are dead before it is written) but never the band spectra, which are filled
  // while they are live
  const size_t ws = (size_t)g.n2 * L.cpitch;
  L.ws_off = 0;
  L.st_off = ws;
  L.db_off = std::max(gsz, ws + adj_stage_elems(g, elem));
  L.tw_off = L.db_off + (size_t)L.rows * (g.K1 + 1) * 2;
  L.total = L.tw_off + 2 * (size_t)(g.n1 + g.n2);
  return L;
}

// First-step accessor of its row transforms: bin k of the row's spectrum (1 - k) D(k)
// from the band's column data db ([row][kx] complex).
template <typename T>
struct RecSpecAcc {
  const T *db;
  T *r0, *r1;
  int stride, row, per, n1, K1;
  bool pair;
  __device__ void load(int k, T &re, T &im) const {
    const int kk = k <= n1 / 2 ? k : n1 - k;
    re = T(0);
    im = T(0);
    if (kk > K1) return;
    const bool neg = k != kk;
    const T *d = db + 2 * (row * per + kk);
    T dr = d[0], di = d[1];
    if (neg) di = -di;
    if (!pair) {
      const T kf = neg ? -T(kk) : T(kk);
      re = dr - kf * dr;
      im = di - kf * di;
    } else {
      T br = d[2 * per], bi = d[2 * per + 1];
      if (neg) bi = -bi;
      re = dr - bi;
      im = di + br;
    }
  }
  __device__ void store(int i, T re, T im) const {
    r0[i * stride] = re;
    r1[i * stride] = im;
  }
};

// The truncated series at one point, if the point's footprint starts in this band.
template <int W, bool POLY>
__device__ __forceinline__ void rec_point(const AdjArgs<float> &a, const float *Guv, int apitch, int band_lo,
                                          int64_t j, float xj, float yj, float hj, float wj, float cx, float cy,
                                          float R, float pr, double (&acc)[3]) {
  using T = float;
  const Geom &g = a.g;
  const T halfw = T(W) / T(2);
  const FineCoord<T> fy = fine_coord<T>(yj, a.s2_hi, a.s2_lo, halfw);
  const int r0 = (fy.i0 & (g.n2 - 1)) - band_lo;    // first footprint row, band-local
  if (r0 < 0 || r0 >= a.band_rows) return;
  const FineCoord<T> fx = fine_coord<T>(xj, a.s1_hi, a.s1_lo, halfw);
  T kx[W];
  T u = 0;
  const float2 *puv = reinterpret_cast<const float2 *>(Guv) + r0 * apitch + (fx.i0 & (g.n1 - 1));
  auto row = [&](T kyv) {
    T su = 0;
#pragma unroll
    for (int dx = 0; dx < W; ++dx) su += kx[dx] * puv[dx].x;
    u += kyv * su;
    puv += apitch;
  };
  if constexpr (POLY) {
    T ky[W];
    es_taps_poly<W>(fx, float(W) * 0.5f, a.es, kx);
    es_taps_poly<W>(fy, float(W) * 0.5f, a.es, ky);
#pragma unroll
    for (int dy = 0; dy < W; ++dy) row(ky[dy]);
  } else {
    const T zsc = T(2) / T(W);
#pragma unroll
    for (int d = 0; d < W; ++d) kx[d] = ker_eval(fx.offset(d) * zsc, a.beta);
#pragma unroll 1
    for (int dy = 0; dy < W; ++dy) row(ker_eval(fy.offset(dy) * zsc, a.beta));
  }
  const double t = (double)(hj * hann_w(a.window_kind, xj, yj, cx, cy, R, pr));
  const double d = t - (double)u;
  acc[0] += d * d;
  acc[1] += t * t;
  acc[2] += (double)wj * t * t;
  if (a.grad_h) a.grad_h[j] = u;
}

// All points of one item; every point is read (its band decides whether it is
// served).  Wave w takes blocks of 256 consecutive points and lane l gathers
// points l, l + 64, l + 128 and l + 192 of a block, so at every step the 64 lanes
// work on 64 consecutive points (overlapping footprints in raster order).  The
// loads run two blocks ahead in three register buffers.  The wider kernels
// (register budget) take one point per thread and step.
template <int W, int NT, bool POLY>
__device__ __forceinline__ void rec_item(const AdjArgs<float> &a, const float *Guv, int apitch, int band_lo,
                                         int64_t begin, int64_t end, float cx, float cy, float R,
                                         double (&acc)[3]) {
  using T = float;
  const T pr = R > T(0) ? T(M_PI) / R : T(0);
  if constexpr (W <= 6) {
    constexpr int U = 4, BLK = 64 * U, NWV = NT / 64;
    struct Pts {
      T x[U], y[U], h[U], w[U];
    };
    const int lane = threadIdx.x & 63;
    const int64_t stride = (int64_t)NWV * BLK;
    auto load = [&](Pts &b, int64_t pb) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int64_t i = pb + u * 64 + lane;
        const int64_t ic = i < end ? i : end - 1;   // past the end: re-read the last point (unused)
        b.x[u] = a.x[ic]; b.y[u] = a.y[ic]; b.h[u] = a.h[ic]; b.w[u] = a.w[ic];
      }
    };
    auto step = [&](const Pts &b, int64_t pb) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int64_t i = pb + u * 64 + lane;
        if (i < end)
          rec_point<W, POLY>(a, Guv, apitch, band_lo, i, b.x[u], b.y[u], b.h[u], b.w[u], cx, cy, R, pr, acc);
      }
    };
    if (begin < end) {
      int64_t p = begin + (int64_t)(threadIdx.x >> 6) * BLK;
      Pts b0, b1, b2;
      load(b0, p);
      load(b1, p + stride);
      for (; p < end; p += 3 * stride) {
        load(b2, p + 2 * stride);
        step(b0, p);
        load(b0, p + 3 * stride);
        step(b1, p + stride);
        load(b1, p + 4 * stride);
        step(b2, p + 2 * stride);
      }
    }
  } else {
    for (int64_t j = begin + threadIdx.x; j < end; j += NT)
      rec_point<W, POLY>(a, Guv, apitch, band_lo, j, a.x[j], a.y[j], a.h[j], a.w[j], cx, cy, R, pr, acc);
  }
}

template <int W, bool POLY>
__global__ __launch_bounds__(ADJ_THREADS) void rec_kernel(AdjArgs<float> a) {
  using T = float;
  constexpr int NT = ADJ_THREADS;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  T *sm = reinterpret_cast<T *>(smem_raw);
  __shared__ int s_item;
  const Geom &g = a.g;
  const RecLayout L = rec_layout(g, W, a.band_rows, sizeof(T));
  const int pitch = L.apitch;
  T *Guv = sm;   // rows of (u, du/dx) pairs, interleaved
  T *db = sm + L.db_off, *ws = sm + L.ws_off;
  const int per = g.K1 + 1;
  // the transforms' twiddles stay in LDS for all items of this workgroup (the
  // barrier at the top of the item loop orders them before first use)
  T *tw1 = sm + L.tw_off, *tw2 = tw1 + 2 * g.n1;
  for (int i = threadIdx.x; i < 2 * g.n1; i += NT) tw1[i] = a.tw1[i];
  for (int i = threadIdx.x; i < 2 * g.n2; i += NT) tw2[i] = a.tw2[i];
  for (;;) {
    if (threadIdx.x == 0) s_item = atomicAdd(a.work_counter, 1);
    __syncthreads();
    const int64_t idx = s_item;
    __syncthreads();
    if (idx >= a.n_items) break;
    const AdjItem it = a.items[idx];
    const T *gc = a.fbar + (int64_t)it.cell * g.N1 * g.N2 * 2;
    const int y0 = it.band * a.band_rows;   // fine row of band-local row 0
    T *st = sm + L.st_off;
    stage_spectrum<T, NT>(a, gc, it.cell, st);
    column_pass<T, NT>(a, st, tw2, T(1), ws, L.cpitch, false, db, L.rows, y0);
    // the (u, du/dx) rows, spectrum (1 - k) D(k)
    float *db0 = db, *db1 = db, *Gy = Guv;
    constexpr bool RECON = true;
    const int n1 = g.n1;
    const int ny_pairs = L.rows / 2;
    const int K1 = g.K1;
    row_ifft_natural<NT, T>(
        n1, RECON ? L.rows : L.rows + ny_pairs, tw1, W - 1,
        [&](int q) {
          RecSpecAcc<T> acc;
          acc.db = q < L.rows ? db0 : db1;
          acc.row = q < L.rows ? q : 2 * (q - L.rows);
          acc.pair = q >= L.rows;
          acc.per = per;
          acc.n1 = n1;
          acc.K1 = K1;
          if (q < L.rows) {
            acc.r0 = Guv + 2 * q * pitch;
            acc.r1 = acc.r0 + 1;
            acc.stride = 2;
          } else {
            acc.r0 = Gy + 2 * (q - L.rows) * pitch;
            acc.r1 = acc.r0 + pitch;
            acc.stride = 1;
          }
          return acc;
        },
        [&](int q) {
          StridedPairAcc<T> acc;
          if (q < L.rows) {
            acc.r0 = Guv + 2 * q * pitch;
            acc.r1 = acc.r0 + 1;
            acc.stride = 2;
          } else {
            acc.r0 = Gy + 2 * (q - L.rows) * pitch;
            acc.r1 = acc.r0 + pitch;
            acc.stride = 1;
          }
          return acc;
        });

    const double *wn = a.windows + 3 * (int64_t)it.cell;
    double acc[3] = {0.0, 0.0, 0.0};
    rec_item<W, NT, POLY>(a, Guv, pitch, y0, it.begin, it.end, T(wn[0]), T(wn[1]), T(wn[2]), acc);
    // the item's three sums, reduced in a fixed order (waves, then lanes)
    __syncthreads();
    double *red = reinterpret_cast<double *>(sm);
    for (int k = 0; k < 3; ++k) {
      double v = acc[k];
      for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
      if ((threadIdx.x & 63) == 0) red[k * (NT / 64) + (threadIdx.x >> 6)] = v;
    }
    __syncthreads();
    if (threadIdx.x < 3) {
      double v = 0.0;
      for (int q = 0; q < NT / 64; ++q) v += red[threadIdx.x * (NT / 64) + q];
      a.rec_part[3 * idx + threadIdx.x] = v;
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    __threadfence();
    const int old = atomicAdd(a.done_counter, 1);
    if (old == (int)gridDim.x - 1) {
      *a.work_counter = 0;
      *a.done_counter = 0;
    }
  }
}

template <int W>
static const void *rec_fn_w(bool poly) {
  if constexpr (W <= ES_MAXW) {
    if (poly) return (const void *)&rec_kernel<W, true>;
  }
  return (const void *)&rec_kernel<W, false>;
}

static const void *rec_fn(int W, bool poly) {
  switch (W) {
    case 4: return rec_fn_w<4>(poly);
    case 6: return rec_fn_w<6>(poly);
    case 8: return rec_fn_w<8>(poly);
    case 10: return rec_fn_w<10>(poly);
    case 12: return rec_fn_w<12>(poly);
    case 14: return rec_fn_w<14>(poly);
    case 16: return rec_fn_w<16>(poly);
    default: return nullptr;
  }
}

// ------------------------------------------------------------------ single-grid adjoint
//
// FP32 plans whose kernel takes the polynomial path: the cell's whole real grid
// of u (the inverse transform of the pre-corrected, Hermitian spectrum) fits
// LDS, and du/dx, du/dy come from the same grid through the derivatives of the
// kernel taps: u(t) = sum_m G_m psi_x psi_y, du/dt_x = sum_m G_m psi_x' psi_y.
// The interpolant's derivative converges more slowly than the interpolant, so
// this path uses its own kernel two cells wider than the forward's (with its
// own deconvolution factors).  One pass per cell: one column transform pass,
// half as many row transforms as rows (real rows in pairs), then the gather.

struct Adj1Layout {
  int rows;      // grid rows stored: n2 + W (the first W - 1 repeated after the last)
  int apitch;    // row pitch: n1 + W - 1 rounded up to even (first W - 1 columns repeated)
  int cpitch;    // column-workspace pitch
  int rsplit;    // compact layout: rows [rsplit, n2) are transformed in the staged batch; 0: not compact
  size_t g_off, ws_off, st_off, db_off, tw_off, total;   // element offsets
};

// The column output db ([n2][K1 + 1] complex) must not overlap the column
// workspace while the column pass writes it.  Compact layout: db ends where the
// grid does, so it shares the grid's last rows; the row transforms then run in
// two batches, rows [0, rsplit) (which lie below db) and rows [rsplit, n2), whose
// first step loads every input before any store (at most one item per thread of
// the NT-thread workgroup).  Otherwise db follows the grid.
__host__ __device__ inline Adj1Layout adj1_layout(const Geom &g, int W, size_t elem, int NT) {
  Adj1Layout L;
  L.rows = g.n2 + W;
  L.apitch = (g.n1 + W - 1 + 1) & ~1;
  L.cpitch = 2 * (g.K1 + 1) + 2;
  L.g_off = 0;
  // the column workspace and the staged spectrum alias the grid (both are dead
  // before the row transforms write it)
  L.ws_off = 0;
  const size_t ws = (size_t)g.n2 * L.cpitch;
  L.st_off = ws;
  const size_t gsz = (size_t)L.rows * L.apitch, wst = ws + adj_stage_elems(g, elem);
  const size_t dbsz = (size_t)g.n2 * (g.K1 + 1) * 2;
  L.rsplit = 0;
  size_t db = gsz > wst ? gsz : wst;
  if (gsz >= dbsz && gsz - dbsz >= ws) {
    const size_t dc = gsz - dbsz;
    int rs = (int)(dc / L.apitch) & ~1;                 // rows [0, rs) end at or below db
    const int items = (g.n2 - rs) / 2 * fft_B(g.n1);    // first-step items of the staged batch
    if (rs >= 2 && rs < g.n2 && items <= NT) {
      L.rsplit = rs;
      db = dc;
    }
  }
  L.db_off = db;
  const size_t end = db + dbsz;
  const size_t top = end > gsz ? end : gsz;
  L.tw_off = top > wst ? top : wst;
  L.total = L.tw_off + 2 * (size_t)(g.n1 + g.n2);
  return L;
}

// First step of the row-pair inverse transforms for pairs [q0, q0 + count) whose
// spectra are read from LDS that the step's own stores overwrite: every item
// loads its A inputs, the workgroup waits, then every item transforms and
// stores (one item per thread, count * B <= NT).  The same arithmetic as
// fft4_step1_swz.
template <int A, int B, int NT, typename Make>
__device__ __forceinline__ void row_step1_staged(int q0, int count, const float *tw, const Make &make1) {
  const int it = threadIdx.x;
  const bool on = it < count * B;
  const int q = q0 + (on ? it / B : 0), b = on ? it % B : 0;
  const auto acc = make1(q);
  float re[A], im[A];
#pragma unroll
  for (int a = 0; a < A; ++a) {
    re[a] = 0.0f;
    im[a] = 0.0f;
    if (on) acc.load(a * B + b, re[a], im[a]);
  }
  __syncthreads();
  if (on) {
    dft_reg<A, true, float>(re, im);
#pragma unroll
    for (int k1 = 0; k1 < A; ++k1) {
      float r = re[k1], i = im[k1];
      if (k1 > 0) {
        const int j = b * k1;
        const float c = tw[2 * j], sn = -tw[2 * j + 1];
        const float nr = r * c - i * sn;
        i = r * sn + i * c;
        r = nr;
      }
      acc.store(k1 * B + (b ^ fft_swz(k1, B)), r, i);
    }
  }
  __syncthreads();
}

// Taps and their derivatives from the mirror-pair polynomials of the taps alone
// (no second set of coefficients, so the kernel's scalar registers hold one
// table).  With P_d(u) = E(s) + u O(s) and s = u^2: dP_d/du = O + 2 u (E' + u O'),
// and the mirror tap W - 1 - d, E - u O, has -O + 2 u (E' - u O'); E' and O'
// (d/ds) come out of the same Horner steps.
// Mirror pair d of the taps and of their u-derivatives: tap d, tap W - 1 - d and
// the two derivatives dP/du, from the pair's coefficients cd at u and s = u^2.
// (With u = 2 (i0 - t + W/2) - 1, d/dt = -2 d/du: the caller's scale carries the
// factor -2, so it is not multiplied into every tap.)
__device__ __forceinline__ void es_pair_dtaps(float u, float s, const float *cd, float &t0, float &t1, float &d0,
                                              float &d1) {
  float e = cd[ES_DEG - 1], o = cd[ES_DEG], de = e, dO = o;
#pragma unroll
  for (int k = ES_DEG - 3; k >= 0; k -= 2) {
    if (k < ES_DEG - 3) {   // (the first step's derivatives are the leading coefficients)
      de = fmaf(de, s, e);
      dO = fmaf(dO, s, o);
    }
    e = fmaf(e, s, cd[k]);
    o = fmaf(o, s, cd[k + 1]);
  }
  t0 = fmaf(u, o, e);
  t1 = fmaf(-u, o, e);
  const float u2 = 2.0f * u;
  d0 = fmaf(u2, fmaf(u, dO, de), o);
  d1 = fmaf(u2, fmaf(-u, dO, de), -o);
}

template <int W>
__device__ __forceinline__ void es_taps_dtaps_poly_v(float v, const EsPoly &cf, float (&out)[W],
                                                     float (&dout)[W]) {
  const float u = 2.0f * v - 1.0f;
  const float s = u * u;
#pragma unroll
  for (int d = 0; d < W / 2; ++d)
    es_pair_dtaps(u, s, cf.c + d * (ES_DEG + 1), out[d], out[W - 1 - d], dout[d], dout[W - 1 - d]);
}

// Holds the two rows' grid values until every read of the pair has returned,
// so the reads are issued together and waited for once (left to itself the
// compiler waited after each read, one LDS round trip per two values).
template <int W>
__device__ __forceinline__ void hold_rows(float (&ra)[W], float (&rb)[W]) {
  if constexpr (W == 8) {
    asm volatile("" : "+v"(ra[0]), "+v"(ra[1]), "+v"(ra[2]), "+v"(ra[3]), "+v"(ra[4]), "+v"(ra[5]), "+v"(ra[6]),
                      "+v"(ra[7]), "+v"(rb[0]), "+v"(rb[1]), "+v"(rb[2]), "+v"(rb[3]), "+v"(rb[4]), "+v"(rb[5]),
                      "+v"(rb[6]), "+v"(rb[7]));
  } else if constexpr (W == 6) {
    asm volatile("" : "+v"(ra[0]), "+v"(ra[1]), "+v"(ra[2]), "+v"(ra[3]), "+v"(ra[4]), "+v"(ra[5]), "+v"(rb[0]),
                      "+v"(rb[1]), "+v"(rb[2]), "+v"(rb[3]), "+v"(rb[4]), "+v"(rb[5]));
  }
}

// An item's point arrays (at its first point) and the plan's constants of the gather.
struct Gather1 {
  const float *x, *y, *h, *w;
  float *gh, *gx, *gy;
  float cx, cy, R, pr;
};

// Element at a 32-bit byte offset of a uniform base (one scalar base, one vector offset).
__device__ __forceinline__ float at_offset(const float *p, unsigned o) {
  return *reinterpret_cast<const float *>(reinterpret_cast<const char *>(p) + o);
}
__device__ __forceinline__ void put_offset(float *p, unsigned o, float v) {
  *reinterpret_cast<float *>(reinterpret_cast<char *>(p) + o) = v;
}

// Gradients at one point: W x W taps of the grid with value and derivative
// weights (row sums with psi_x and psi_x', then combined with psi_y, psi_y'),
// then the chain rule through the strength as in gather_point.  ALL: all three
// gradients are wanted (no tests per point).
template <int W, bool ALL>
__device__ __forceinline__ void gather1_point(const AdjArgs<float> &a, const Gather1 &q, const float *G, int apitch,
                                              unsigned o, float xj, float yj, float hj, float wj) {
  const float halfw = float(W) * 0.5f;
  const FineCoord<float> fx = fine_coord<float>(xj, a.s1_hi, a.s1_lo, halfw);
  const FineCoord<float> fy = fine_coord<float>(yj, a.s2_hi, a.s2_lo, halfw);
  const float vx = tap_v(fx, halfw), vy = tap_v(fy, halfw);
  float kx[W], kxd[W];
  es_taps_dtaps_poly_v<W>(vx, a.es, kx, kxd);
  const float uyv = 2.0f * vy - 1.0f, syv = uyv * uyv;
  const float *p = G + (fy.i0 & (a.g.n2 - 1)) * apitch + (fx.i0 & (a.g.n1 - 1));
  float u = 0.0f, ux = 0.0f, uy = 0.0f;
  // rows in mirror pairs (d, W - 1 - d), whose y taps come from one polynomial pair
#pragma unroll
  for (int d = 0; d < W / 2; ++d) {
    const float *pa = p + d * apitch, *pb = p + (W - 1 - d) * apitch;
    float ra[W], rb[W];
#pragma unroll
    for (int dx = 0; dx < W; ++dx) {
      ra[dx] = pa[dx];
      rb[dx] = pb[dx];
    }
    float ta, tb, da, db;
    es_pair_dtaps(uyv, syv, a.es.c + d * (ES_DEG + 1), ta, tb, da, db);
    hold_rows<W>(ra, rb);
    float sa = kx[0] * ra[0], sda = kxd[0] * ra[0], sb = kx[0] * rb[0], sdb = kxd[0] * rb[0];
#pragma unroll
    for (int dx = 1; dx < W; ++dx) {
      sa = fmaf(kx[dx], ra[dx], sa);
      sda = fmaf(kxd[dx], ra[dx], sda);
      sb = fmaf(kx[dx], rb[dx], sb);
      sdb = fmaf(kxd[dx], rb[dx], sdb);
    }
    u = fmaf(ta, sa, u);
    ux = fmaf(ta, sda, ux);
    uy = fmaf(da, sa, uy);
    u = fmaf(tb, sb, u);
    ux = fmaf(tb, sdb, ux);
    uy = fmaf(db, sb, uy);
  }
  // the derivative sums are formed here, in the row loop, not sunk into the
  // branch that stores them (which kept all W x W grid values live)
  asm volatile("" : "+v"(ux), "+v"(uy));
  ux *= a.dsx;   // -2 n1 / (2 pi): d/dt of the fine coordinate, d/du = -2 d/dt
  uy *= a.dsy;
  float dWx, dWy;
  const float Wv = hann_wg(a.window_kind, xj, yj, q.cx, q.cy, q.R, q.pr, dWx, dWy);
  if (ALL || q.gh) put_offset(q.gh, o, wj * Wv * u);
  if (ALL || q.gx || q.gy) {
    const float wh = wj * hj;
    if (ALL || q.gx) put_offset(q.gx, o, wh * (dWx * u + Wv * ux));
    if (ALL || q.gy) put_offset(q.gy, o, wh * (dWy * u + Wv * uy));
  }
}

// All points of one item: wave w takes blocks of 64 consecutive points, one per
// lane (so the 64 lanes of a step read overlapping footprints of raster-ordered
// points); each lane's next point is loaded while the current one is gathered.
// (Four points per lane and block, picked by a run-time index, had put the
// buffers in scratch memory: 16 bytes per point written and read back.)  Indices
// are 32-bit offsets from the item's first point: with 64-bit point indices each
// access formed its own address, and with the kernel's arguments held from its start
// 56 of the loop's 473 vector instructions per point read spilled scalar registers
// back; both gone, 8,192 triangles of 3.3e8 samples went from 3.83 to 3.41 ms.
template <int W, int NT, bool ALL>
__device__ __forceinline__ void gather1_item(const AdjArgs<float> &a, const Gather1 &q, const float *G, int apitch,
                                             int n) {
  constexpr int stride = NT;
  struct Pt {
    float x, y, h, w;
  };
  auto load = [&](Pt &b, int i) {
    const unsigned o = 4u * (unsigned)(i < n ? i : n - 1);   // past the end: re-read the last point (unused)
    b.x = at_offset(q.x, o); b.y = at_offset(q.y, o); b.h = at_offset(q.h, o); b.w = at_offset(q.w, o);
  };
  int i = threadIdx.x;
  Pt b0, b1;
  load(b0, i);
  for (; i - (int)(threadIdx.x & 63) < n; i += 2 * stride) {
    load(b1, i + stride);
    if (i < n) gather1_point<W, ALL>(a, q, G, apitch, 4u * (unsigned)i, b0.x, b0.y, b0.h, b0.w);
    load(b0, i + 2 * stride);
    if (i + stride < n) gather1_point<W, ALL>(a, q, G, apitch, 4u * (unsigned)(i + stride), b1.x, b1.y, b1.h, b1.w);
  }
}

// Four waves per SIMD: two 512-thread workgroups per CU with the compact layout
// (each thread then within 128 VGPRs).
template <int W, int NT>
__global__ __launch_bounds__(NT, (NT == 512 ? 4 : 1)) void adj1_kernel(AdjArgs<float>) {
  const AdjArgs<float> &a = fresh_args<AdjArgs<float>>();
  extern __shared__ __align__(16) unsigned char smem_raw[];
  float *sm = reinterpret_cast<float *>(smem_raw);
  __shared__ int s_item;
  const Geom &g = a.g;
  const Adj1Layout L = adj1_layout(g, W, sizeof(float), NT);
  float *G = sm + L.g_off, *ws = sm + L.ws_off, *st = sm + L.st_off, *db = sm + L.db_off;
  float *tw1 = sm + L.tw_off, *tw2 = tw1 + 2 * g.n1;
  const int per = g.K1 + 1, pitch = L.apitch;
  for (int i = threadIdx.x; i < 2 * g.n1; i += NT) tw1[i] = a.tw1[i];
  for (int i = threadIdx.x; i < 2 * g.n2; i += NT) tw2[i] = a.tw2[i];
  for (;;) {
    if (threadIdx.x == 0) s_item = atomicAdd(a.work_counter, 1);
    __syncthreads();
    const int64_t idx = s_item;
    __syncthreads();
    if (idx >= a.n_items) break;
    const AdjItem it = a.items[idx];
    const float *gc = a.fbar + (int64_t)it.cell * g.N1 * g.N2 * 2;
    const float two_lam = a.keep ? float(2.0 * (a.lam ? a.lam[it.cell] : 1.0)) : 1.0f;
    stage_spectrum<float, NT>(a, gc, it.cell, st);
    // columns kx = 0 .. K1 of the pre-corrected spectrum, inverse transformed along y
    column_pass<float, NT>(a, st, tw2, two_lam, ws, L.cpitch, false, db, g.n2, 0);
    // rows in pairs: Z(k) = D_2q(k) + i D_2q+1(k) gives rows 2q and 2q + 1 as its real
    // and imaginary parts (both rows' spectra are Hermitian)
    const int n1 = g.n1, K1 = g.K1;
    auto make1 = [&](int q) {
      RowSpecAcc<float> acc;
      acc.db = db;
      acc.row = 2 * q;
      acc.pair = true;
      acc.per = per;
      acc.n1 = n1;
      acc.K1 = K1;
      acc.r0 = G + 2 * q * pitch;
      acc.r1 = acc.r0 + pitch;
      acc.stride = 1;
      return acc;
    };
    auto make2 = [&](int q) {
      StridedPairAcc<float> acc;
      acc.r0 = G + 2 * q * pitch;
      acc.r1 = acc.r0 + pitch;
      acc.stride = 1;
      return acc;
    };
    if (L.rsplit == 0) {
      row_ifft_natural<NT, float>(n1, g.n2 / 2, tw1, W - 1, make1, make2);
    } else {
      // rows below db first, then the rows that share its space
      const int qs = L.rsplit / 2, qn = g.n2 / 2 - qs;
      row_ifft_natural<NT, float>(n1, qs, tw1, W - 1, make1, make2);
      switch (n1) {
        case 16: row_step1_staged<4, 4, NT>(qs, qn, tw1, make1); break;
        case 32: row_step1_staged<8, 4, NT>(qs, qn, tw1, make1); break;
        case 64: row_step1_staged<8, 8, NT>(qs, qn, tw1, make1); break;
        default: row_step1_staged<16, 8, NT>(qs, qn, tw1, make1); break;
      }
      const int A2 = fft_A(n1), la = fft_logA(n1);
      for (int it = threadIdx.x; it < qn * A2; it += NT) {
        const int q = qs + (it >> la), k1 = it & (A2 - 1);
        switch (n1) {
          case 16: row_step2_natural<4, 4, float>(make2(q), k1, n1, W - 1); break;
          case 32: row_step2_natural<8, 4, float>(make2(q), k1, n1, W - 1); break;
          case 64: row_step2_natural<8, 8, float>(make2(q), k1, n1, W - 1); break;
          default: row_step2_natural<16, 8, float>(make2(q), k1, n1, W - 1); break;
        }
      }
      __syncthreads();
    }
    // the first W - 1 rows again after the last (with their repeated columns)
    for (int i = threadIdx.x; i < (W - 1) * pitch; i += NT) G[g.n2 * pitch + i] = G[i];
    __syncthreads();
    {
      const AdjArgs<float> &b = fresh_args<AdjArgs<float>>();
      const double *wn = b.windows + 3 * (int64_t)it.cell;
      Gather1 q;
      q.x = b.x + it.begin; q.y = b.y + it.begin; q.h = b.h + it.begin; q.w = b.w + it.begin;
      q.gh = b.grad_h ? b.grad_h + it.begin : nullptr;
      q.gx = b.grad_x ? b.grad_x + it.begin : nullptr;
      q.gy = b.grad_y ? b.grad_y + it.begin : nullptr;
      q.cx = float(wn[0]); q.cy = float(wn[1]); q.R = float(wn[2]);
      q.pr = q.R > 0.0f ? float(M_PI) / q.R : 0.0f;
      const int n = (int)(it.end - it.begin);
      if (n > 0) {
        if (q.gh && q.gx && q.gy) gather1_item<W, NT, true>(b, q, G, pitch, n);
        else gather1_item<W, NT, false>(b, q, G, pitch, n);
      }
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    __threadfence();
    const int old = atomicAdd(a.done_counter, 1);
    if (old == (int)gridDim.x - 1) {
      *a.work_counter = 0;
      *a.done_counter = 0;
    }
  }
}

static const void *adj1_fn(int W, int threads) {
  if (W == 6) return threads == 512 ? (const void *)&adj1_kernel<6, 512> : (const void *)&adj1_kernel<6, 1024>;
  if (W == 8) return threads == 512 ? (const void *)&adj1_kernel<8, 512> : (const void *)&adj1_kernel<8, 1024>;
  return nullptr;
}

static hipError_t launch_adj1(const AdjArgs<float> &a, int W, int blocks, int threads, size_t lds, hipStream_t s) {
  const void *fn = adj1_fn(W, threads);
  if (!fn) return hipErrorInvalidValue;
  void *args[] = {const_cast<AdjArgs<float> *>(&a)};
  return hipLaunchKernel(fn, dim3(blocks), dim3(threads), args, lds, s);
}

// ------------------------------------------------------------------ host side

enufft_status record_start(enufft_plan_t p, int kind, hipEvent_t *ev);
enufft_status record_stop(enufft_plan_t p, int kind, hipEvent_t start);
template <typename T>
void split_scale(int n, T *hi, T *lo);

// Bands per cell: the fewest row bands whose grid planes fit one workgroup's LDS.
static int choose_bands(const Geom &g, int W, size_t elem, bool recon, size_t lds_max, int *band_rows, size_t *lds) {
  if (W & 1) return 0;   // rows are transformed in pairs: band rows must be even
  for (int B = 1; B <= g.n2 / 2; B <<= 1) {
    const int R = g.n2 / B;
    const size_t bytes = recon && elem == 4 ? rec_layout(g, W, R, elem).total * elem
                                            : band_layout(g, W, R, elem, recon, ADJ_THREADS).total;
    if (bytes <= lds_max) {
      *band_rows = R;
      *lds = bytes;
      return B;
    }
  }
  return 0;
}

// Work list of the cells [c0, c1): every (cell, band) pair, cells above the chunk
// target cut into point chunks (gathers need no merge), longest first.  A chunk
// serves at least `least` points of its band: fewer cost less than the band's
// row transforms.
static void build_adj_items(enufft_plan_t p, int64_t c0, int64_t c1, int slots, int B, int64_t least,
                            std::vector<AdjItem> &items) {
  const int64_t Q = p->offsets[c1] - p->offsets[c0];
  const int64_t per = (int64_t)p->adj_items_per_slot * std::max(1, slots);
  // (at most 2^28 points: the gathers' offsets inside an item are 32-bit)
  const int64_t T = std::min<int64_t>(std::max<int64_t>(least * B, (Q * B + per - 1) / per), int64_t(1) << 28);
  const size_t first = items.size();
  for (int64_t c = c0; c < c1; ++c) {
    const int64_t a = p->offsets[c], b = p->offsets[c + 1];
    const int64_t q = b - a;
    if (q == 0) continue;
    const int64_t nch = std::max<int64_t>(1, (q + T - 1) / T);
    for (int band = 0; band < B; ++band)
      for (int64_t i = 0; i < nch; ++i)
        items.push_back(AdjItem{a + q * i / nch, a + q * (i + 1) / nch, (int32_t)c, band, 0, 0});
  }
  std::stable_sort(items.begin() + first, items.end(), [](const AdjItem &x, const AdjItem &y) {
    return (x.end - x.begin) > (y.end - y.begin);
  });
}

// Release the adjoint schedules so the next call rebuilds them (autotuner: while the
// plan is made, before any reconstruction).
void adj_reset(enufft_plan_t p) {
  dev_release(p, &p->adj.d_items, std::max<size_t>(16, p->adj.items.size() * sizeof(AdjItem)));
  p->adj = AdjSched{};
  dev_release(p, &p->d_adj1_items, std::max<size_t>(16, p->adj1_items.size() * sizeof(AdjItem)));
  p->adj1_items.clear();
}

// While the caller's stream is being captured, allocations and uploads of a first call
// would be refused (a capture records launches): they run outside it, the uploads on a
// stream of their own (the default stream would join the capture).
struct OutsideCapture {
  hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
  OutsideCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
  ~OutsideCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
};

static hipError_t outside_copy(enufft_plan_t p, void *d, const void *src, size_t bytes) {
  hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(p->stream, &st) != hipSuccess) (void)hipGetLastError();
  if (st == hipStreamCaptureStatusNone) return hipMemcpy(d, src, bytes, hipMemcpyHostToDevice);
  hipStream_t s = nullptr;
  hipError_t e = hipStreamCreateWithFlags(&s, hipStreamNonBlocking);
  if (e == hipSuccess) e = hipMemcpyAsync(d, src, bytes, hipMemcpyHostToDevice, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  if (s) (void)hipStreamDestroy(s);
  return e;
}

// Device allocation recorded in the plan's workspace (released with the plan).
static enufft_status adj_alloc(enufft_plan_t p, void **d, size_t bytes, const char *what) {
  hipError_t e = hipMalloc(d, std::max<size_t>(16, bytes));
  if (e != hipSuccess) {
    *d = nullptr;
    (void)hipGetLastError();   // (not left for the check of a later launch)
    p->last_error = std::string(what) + " allocation failed";
    return ENUFFT_ENOMEM;
  }
  p->allocations.push_back(*d);
  p->workspace_bytes += (int64_t)std::max<size_t>(16, bytes);
  return ENUFFT_OK;
}

static enufft_status adj_upload(enufft_plan_t p, void **d, const void *src, size_t bytes, const char *what) {
  enufft_status st = adj_alloc(p, d, bytes, what);
  if (st != ENUFFT_OK || bytes == 0) return st;
  const hipError_t e = outside_copy(p, *d, src, bytes);
  if (e != hipSuccess) {
    p->last_error = std::string(what) + " upload: " + hipGetErrorString(e);
    p->faulted = true;
    return ENUFFT_EDEVICE;
  }
  return ENUFFT_OK;
}

// Workgroups of `fn` the device holds at once, or 0.
static int adj_slots(enufft_plan_t p, const void *fn, int threads, size_t lds) {
  int per_cu = 0;
  if (!fn || hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess) return 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, threads, lds) != hipSuccess) return 0;
  return per_cu * p->n_cu;
}

static const void *band_fn(enufft_plan_t p, bool recon) {
  if (recon && p->prec == ENUFFT_F32) return rec_fn(p->W, p->es.on != 0);
  return p->prec == ENUFFT_F64 ? adj_fn_w<double>(p->W, p->es64.on != 0, recon)
                               : adj_fn_w<float>(p->W, p->es.on != 0, recon);
}

// The column spectra of one launch take at most this much device memory; larger
// batches run in groups of cells, one pair of launches each.
constexpr size_t ADJ_COLS_CAP = (size_t)512 << 20;

static size_t cols_per_cell(enufft_plan_t p, int nset) {
  return (size_t)nset * p->geom.n2 * (p->geom.K1 + 1) * 2 * p->elem;
}

// The buffer of the column spectra, one for the gradients and the reconstruction (both
// run on the plan's stream and share its work counters).  Where the device or
// ENUFFT_ALLOC_CAP_MB leaves less room the groups get smaller, down to one cell.
static enufft_status cols_prepare(enufft_plan_t p) {
  if (p->d_adj_cols) return ENUFFT_OK;
  const size_t per_cell = cols_per_cell(p, 2);
  const int64_t room = std::min<int64_t>((int64_t)ADJ_COLS_CAP, workspace_room(p));
  int64_t group = std::max<int64_t>(1, std::min<int64_t>(p->n_cells, room / (int64_t)per_cell));
  for (;; group = (group + 1) / 2) {
    const enufft_status st = adj_alloc(p, &p->d_adj_cols, per_cell * (size_t)group, "adjoint column spectra");
    if (st == ENUFFT_OK) p->adj_cols_bytes = per_cell * (size_t)group;
    if (st == ENUFFT_OK || group == 1) return st;
  }
}

// Set up a banded schedule on first use (the gradients' or the reconstruction's).
static enufft_status band_prepare(enufft_plan_t p, AdjSched *s, bool recon) {
  if (s->ready) return ENUFFT_OK;
  AdjSched n;
  int B = choose_bands(p->geom, p->W, p->elem, recon, p->lds_limit, &n.band_rows, &n.lds);
  if (B == 0) {
    p->last_error = "adjoint: fine-grid bands do not fit in LDS";
    return ENUFFT_EUNSUPPORTED;
  }
  // more bands than the minimum (autotuner choice): smaller LDS footprint per item
  for (int m = recon ? 1 : p->adj_band_mult; m > 1 && p->geom.n2 / (B * 2) >= 2; m >>= 1) {
    B *= 2;
    n.band_rows = p->geom.n2 / B;
    n.lds = band_layout(p->geom, p->W, n.band_rows, p->elem, recon, ADJ_THREADS).total;
  }
  n.bands = B;
  // (the FP32 reconstruction's items transform their own columns)
  const bool own = recon && p->prec == ENUFFT_F32;
  const int slots = adj_slots(p, band_fn(p, recon), ADJ_THREADS, n.lds);
  if (slots < 1) {
    p->last_error = "adjoint kernel cannot be resident";
    return ENUFFT_EDEVICE;
  }
  enufft_status st = own ? ENUFFT_OK : cols_prepare(p);
  if (st != ENUFFT_OK) return st;
  const int64_t fit = own ? p->n_cells : (int64_t)(p->adj_cols_bytes / cols_per_cell(p, recon ? 1 : 2));
  const int64_t group = std::max<int64_t>(1, std::min<int64_t>(p->n_cells, fit));
  for (int64_t c = 0; c < p->n_cells; c += group) {
    n.cell0.push_back(c);
    n.first.push_back((int64_t)n.items.size());
    const int64_t least = p->prec == ENUFFT_F64 ? 512 : own ? 16384 / B : 8192;
    build_adj_items(p, c, std::min(p->n_cells, c + group), slots, B, least, n.items);
  }
  n.cell0.push_back(p->n_cells);
  n.first.push_back((int64_t)n.items.size());
  n.slots = slots;
  st = adj_upload(p, &n.d_items, n.items.data(), n.items.size() * sizeof(AdjItem), "adjoint item");
  if (st != ENUFFT_OK) return st;
  n.ready = true;
  *s = n;
  return ENUFFT_OK;
}

// Device copy of the plan's cell offsets (point sort, geometry, reconstruction), made
// on first use.
enufft_status cell_offsets(enufft_plan_t p) {
  if (p->d_cell_off) return ENUFFT_OK;
  const OutsideCapture outside;
  return adj_upload(p, &p->d_cell_off, p->offsets.data(), p->offsets.size() * sizeof(int64_t), "cell offsets");
}

// Large-cell plans offer the mesh geometry on the grids they have always offered it on,
// up to 256 per axis, about: those where a row band of two rows with its cell's column
// workspace, staged spectrum and band spectra would fit one workgroup's LDS.  (The
// geometry itself needs the cell offsets and its bins only.)
enufft_status geometry_supported(enufft_plan_t p) {
  if (!p->big) return ENUFFT_OK;
  const Geom &g = p->geom;
  for (int R = g.n2; R >= 2; R >>= 1) {
    const size_t rows = (size_t)R + p->W, apitch = (size_t)((g.n1 + p->W) & ~1), per = g.K1 + 1;
    const size_t cols = (size_t)g.n2 * (2 * per + 2) + adj_stage_elems(g, p->elem);
    const size_t total = std::max(3 * rows * apitch, cols) + 4 * rows * per + 2 * (size_t)(g.n1 + g.n2);
    if (total * p->elem <= p->lds_limit) return ENUFFT_OK;
  }
  p->last_error = "enufft_cell_geometry: not offered for a large-cell plan of this fine grid";
  return ENUFFT_EUNSUPPORTED;
}

// Lazily set up the adjoint schedule on first use.
enufft_status adj_prepare(enufft_plan_t p) {
  if (p->adj1 ? p->d_adj1_items != nullptr : p->adj.ready) return ENUFFT_OK;
  const OutsideCapture outside;
  if (!p->adj1) return band_prepare(p, &p->adj, false);
  // single-grid adjoint: one item per cell (or chunk of a large cell), no bands;
  // 512 threads, so two workgroups fit a CU with the compact layout
  if (const char *ev = std::getenv("ENUFFT_ADJ1_THREADS")) p->adj1_threads = std::atoi(ev) == 1024 ? 1024 : 512;
  p->adj1_lds = adj1_layout(p->geom, p->adj1_W, sizeof(float), p->adj1_threads).total * sizeof(float);
  const int slots = adj_slots(p, adj1_fn(p->adj1_W, p->adj1_threads), p->adj1_threads, p->adj1_lds);
  if (slots < 1) {
    p->last_error = "single-grid adjoint kernel cannot be resident";
    return ENUFFT_EDEVICE;
  }
  p->adj1_items.clear();
  build_adj_items(p, 0, p->n_cells, slots, 1, 16384, p->adj1_items);
  p->adj1_blocks = (int)std::min<int64_t>(slots, std::max<int64_t>(1, (int64_t)p->adj1_items.size()));
  void *d = nullptr;
  enufft_status st =
      adj_upload(p, &d, p->adj1_items.data(), p->adj1_items.size() * sizeof(AdjItem), "adjoint item");
  if (st == ENUFFT_OK) p->d_adj1_items = d;
  return st;
}

// The reconstruction's schedule, with the items of each cell, ascending (a cell's
// item partials are summed in this fixed order).
static enufft_status rec_prepare(enufft_plan_t p) {
  if (p->d_rec_part) return ENUFFT_OK;
  const OutsideCapture outside;
  enufft_status st = band_prepare(p, &p->rec, true);
  if (st != ENUFFT_OK) return st;
  const std::vector<AdjItem> &items = p->rec.items;
  std::vector<int64_t> coff(p->n_cells + 1, 0);
  for (const AdjItem &it : items) ++coff[it.cell + 1];
  for (int64_t c = 0; c < p->n_cells; ++c) coff[c + 1] += coff[c];
  std::vector<int32_t> citems(items.size(), 0);
  {
    std::vector<int64_t> pos(coff.begin(), coff.end() - 1);
    for (size_t i = 0; i < items.size(); ++i) citems[pos[items[i].cell]++] = (int32_t)i;
  }
  if (!p->d_cell_items)
    st = adj_upload(p, &p->d_cell_items, citems.data(), citems.size() * sizeof(int32_t), "cell item list");
  if (st == ENUFFT_OK && !p->d_cell_item_off)
    st = adj_upload(p, &p->d_cell_item_off, coff.data(), coff.size() * sizeof(int64_t), "cell item offsets");
  if (st == ENUFFT_OK) st = cell_offsets(p);
  if (st == ENUFFT_OK)
    st = adj_alloc(p, &p->d_rec_part, std::max<size_t>(1, items.size()) * 3 * sizeof(double),
                   "reconstruction partials");
  return st;
}

template <typename T>
AdjArgs<T> make_adj_args(enufft_plan_t p, const void *x, const void *y, const void *h, const void *w,
                         const void *fbar, void *gh, void *gx, void *gy) {
  AdjArgs<T> a{};
  a.x = (const T *)x; a.y = (const T *)y; a.h = (const T *)h; a.w = (const T *)w;
  a.fbar = (const T *)fbar;
  a.keep = nullptr;
  a.lam = nullptr;
  a.grad_h = (T *)gh; a.grad_x = (T *)gx; a.grad_y = (T *)gy;
  a.work_counter = p->d_counters + 2;
  a.done_counter = p->d_counters + 3;
  a.windows = (const double *)p->d_windows;
  a.window_kind = p->window_kind;
  a.decon_x = (const T *)p->d_decon_x; a.decon_y = (const T *)p->d_decon_y;
  a.tw1 = (const T *)p->d_tw1; a.tw2 = (const T *)p->d_tw2;
  a.beta = (T)p->beta;
  split_scale<T>(p->n1, &a.s1_hi, &a.s1_lo);
  split_scale<T>(p->n2, &a.s2_hi, &a.s2_lo);
  a.es = p->es;
  if constexpr (sizeof(T) == 8) a.es64 = p->es64;
  else a.es64.on = 0;
  a.g = p->geom;
  return a;
}

// The banded adjoint (rec_part set: the reconstruction): per group of cells, the
// column transforms, then the band items.
template <typename T>
static hipError_t launch_band(enufft_plan_t p, AdjArgs<T> a, const AdjSched &s) {
  const bool recon = a.rec_part != nullptr;
  const void *fn = band_fn(p, recon);
  const int nset = recon ? 1 : 2, ngrp = adj_col_groups(a.g), cg = (a.g.K1 + 1 + ngrp - 1) / ngrp;
  const size_t lds_cols = ((size_t)a.g.n2 * (2 * cg + 2) + 2 * (size_t)a.g.n2) * sizeof(T);
  a.band_rows = s.band_rows;
  a.cols = (T *)p->d_adj_cols;
  double *part = a.rec_part;
  for (size_t q = 0; q + 1 < s.cell0.size(); ++q) {
    a.items = (const AdjItem *)s.d_items + s.first[q];
    a.n_items = s.first[q + 1] - s.first[q];
    if (a.n_items == 0) continue;
    a.cell0 = (int)s.cell0[q];
    a.rec_part = recon ? part + 3 * s.first[q] : nullptr;
    const int64_t nb = (s.cell0[q + 1] - s.cell0[q]) * nset * ngrp;
    hipError_t e = hipSuccess;
    if (!(recon && sizeof(T) == 4)) {
      hipLaunchKernelGGL(adj_cols_kernel<T>, dim3((unsigned)nb), dim3(ADJ_COLS_THREADS), lds_cols, p->stream, a,
                         nset);
      e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
    void *args[] = {&a};
    e = hipLaunchKernel(fn, dim3((unsigned)std::min<int64_t>(s.slots, a.n_items)), dim3(ADJ_THREADS), args, s.lds,
                        p->stream);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace enufft

namespace enufft {
enufft_status adjoint_common(enufft_plan_t p, const char *fn, const void *x, const void *y, const void *h,
                             const void *w, const void *fin, const uint8_t *keep, const double *lam, void *grad_h,
                             void *grad_x, void *grad_y) {
  if (!p) return ENUFFT_EINVAL;
  if (p->faulted) {
    p->last_error = std::string(fn) + ": plan unusable after a device fault";
    return ENUFFT_ESTATE;
  }
  if (p->n_cells == 0 || p->n_points == 0) return ENUFFT_OK;
  if (!fin) {
    p->last_error = std::string(fn) + ": null coefficient input";
    return ENUFFT_EINVAL;
  }
  if (!x || !y || !h || !w) {   // every kernel reads all four arrays
    p->last_error = std::string(fn) + ": null point array";
    return ENUFFT_EINVAL;
  }
  if (!grad_h && !grad_x && !grad_y) return ENUFFT_OK;
  hipEvent_t ev;
  if (p->big) {
    enufft_status st = record_start(p, 2, &ev);
    if (st != ENUFFT_OK) return st;
    st = big_adjoint(p, x, y, h, w, fin, keep, lam, grad_h, grad_x, grad_y);
    if (st != ENUFFT_OK) return st;
    return record_stop(p, 2, ev);
  }
  enufft_status st = adj_prepare(p);
  if (st != ENUFFT_OK) return st;
  st = record_start(p, 2, &ev);
  if (st != ENUFFT_OK) return st;
  hipError_t e;
  if (p->prec == ENUFFT_F64) {
    auto a = make_adj_args<double>(p, x, y, h, w, fin, grad_h, grad_x, grad_y);
    a.keep = keep;
    a.lam = lam;
    e = launch_band<double>(p, a, p->adj);
  } else if (p->adj1) {
    auto a = make_adj_args<float>(p, x, y, h, w, fin, grad_h, grad_x, grad_y);
    a.keep = keep;
    a.lam = lam;
    a.items = (const AdjItem *)p->d_adj1_items;
    a.n_items = (int64_t)p->adj1_items.size();
    a.decon_x = (const float *)p->d_adj1_decon_x;
    a.decon_y = (const float *)p->d_adj1_decon_y;
    a.es = p->adj1_es;
    a.dsx = (float)(-2.0 * p->n1 / (2.0 * M_PI));   // dt/dx times du/dt of the tap polynomials
    a.dsy = (float)(-2.0 * p->n2 / (2.0 * M_PI));
    e = launch_adj1(a, p->adj1_W, p->adj1_blocks, p->adj1_threads, p->adj1_lds, p->stream);
  } else {
    auto a = make_adj_args<float>(p, x, y, h, w, fin, grad_h, grad_x, grad_y);
    a.keep = keep;
    a.lam = lam;
    e = launch_band<float>(p, a, p->adj);
  }
  if (e != hipSuccess) {
    p->last_error = std::string(fn) + " launch: " + hipGetErrorString(e);
    p->faulted = true;
    return ENUFFT_EDEVICE;
  }
  return record_stop(p, 2, ev);
}
}  // namespace enufft

extern "C" enufft_status enufft_type1_adjoint(enufft_plan_t p, const void *x, const void *y, const void *h,
                                              const void *w, const void *fbar, void *grad_h, void *grad_x,
                                              void *grad_y) {
  return enufft::adjoint_common(p, "enufft_type1_adjoint", x, y, h, w, fbar, nullptr, nullptr, grad_h, grad_x,
                                grad_y);
}

extern "C" enufft_status enufft_retained_power_adjoint(enufft_plan_t p, const void *x, const void *y,
                                                       const void *h, const void *w, const void *f,
                                                       const uint8_t *keep, const double *lam, void *grad_h,
                                                       void *grad_x, void *grad_y) {
  if (p && !keep) {
    p->last_error = "enufft_retained_power_adjoint: null keep";
    return ENUFFT_EINVAL;
  }
  return enufft::adjoint_common(p, "enufft_retained_power_adjoint", x, y, h, w, f, keep, lam, grad_h, grad_x,
                                grad_y);
}

// ------------------------------------------------------------------ reconstruction

namespace enufft {

// Per cell: the sums over its items' partials (fixed order) and the spectral
// sums of Parseval's identity over the modes k != 0, all of them and the kept
// ones (a fixed-order tree over 256 threads), then the diagnostics.
template <typename T>
__global__ __launch_bounds__(256) void rec_finalize_kernel(const T *coef, const uint8_t *keep, const double *area,
                                                           const double *part, const int32_t *cell_items,
                                                           const int64_t *cell_item_off, const int64_t *cell_off,
                                                           Geom g, double *diag) {
  __shared__ double s_all[256], s_kept[256];
  const int64_t c = blockIdx.x;
  const int M = g.N1 * g.N2;
  const T *cc = coef + 2 * (int64_t)M * c;
  const uint8_t *kc = keep ? keep + (int64_t)M * c : nullptr;
  double sa = 0.0, sk = 0.0;
  for (int m = threadIdx.x; m < M; m += 256) {
    const int r = m / g.N1, i = m - r * g.N1;
    if (g.lo1 + i == 0 && g.lo2 + r == 0) continue;
    const double re = (double)cc[2 * m], im = (double)cc[2 * m + 1];
    const double p2 = re * re + im * im;
    sa += p2;
    if (!kc || kc[m]) sk += p2;
  }
  s_all[threadIdx.x] = sa;
  s_kept[threadIdx.x] = sk;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) {
      s_all[threadIdx.x] += s_all[threadIdx.x + o];
      s_kept[threadIdx.x] += s_kept[threadIdx.x + o];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    double e2 = 0.0, t2 = 0.0, wt2 = 0.0;
    for (int64_t q = cell_item_off[c]; q < cell_item_off[c + 1]; ++q) {
      const int64_t it = cell_items[q];
      e2 += part[3 * it];
      t2 += part[3 * it + 1];
      wt2 += part[3 * it + 2];
    }
    const double A = area ? area[c] : 1.0;
    double *d = diag + 8 * c;
    d[0] = (double)(cell_off[c + 1] - cell_off[c]);
    d[1] = e2;
    d[2] = t2;
    d[3] = wt2 / A;
    d[4] = s_all[0];
    d[5] = s_kept[0];
    d[6] = t2 > 0.0 ? sqrt(e2 / t2) : 0.0;
    d[7] = d[3] > 0.0 ? d[4] / d[3] : 0.0;
  }
}

}  // namespace enufft

extern "C" enufft_status enufft_reconstruct(enufft_plan_t p, const void *x, const void *y, const void *h,
                                            const void *w, const void *coef, const uint8_t *keep,
                                            const double *area, void *h_rec, double *diag) {
  using namespace enufft;
  if (!p) return ENUFFT_EINVAL;
  if (p->faulted) {
    p->last_error = "enufft_reconstruct: plan unusable after a device fault";
    return ENUFFT_ESTATE;
  }
  if (p->big) {
    p->last_error = "enufft_reconstruct: not implemented for large-cell plans (mode boxes above 64 per axis)";
    return ENUFFT_EUNSUPPORTED;
  }
  if (p->n_cells == 0) return ENUFFT_OK;
  if (!coef || !diag) {
    p->last_error = "enufft_reconstruct: null coefficients or diagnostics";
    return ENUFFT_EINVAL;
  }
  if (p->n_points > 0 && (!x || !y || !h || !w)) {
    p->last_error = "enufft_reconstruct: null point array";
    return ENUFFT_EINVAL;
  }
  enufft_status st = rec_prepare(p);
  if (st != ENUFFT_OK) return st;
  hipError_t e = hipSuccess;
  if (p->n_points > 0) {
    if (p->prec == ENUFFT_F64) {
      auto a = make_adj_args<double>(p, x, y, h, w, coef, h_rec, nullptr, nullptr);
      a.keep = keep;
      a.decon_x = (const double *)p->d_decon_x1;
      a.rec_part = (double *)p->d_rec_part;
      e = launch_band<double>(p, a, p->rec);
    } else {
      auto a = make_adj_args<float>(p, x, y, h, w, coef, h_rec, nullptr, nullptr);
      a.keep = keep;
      a.decon_x = (const float *)p->d_decon_x1;
      a.rec_part = (double *)p->d_rec_part;
      e = launch_band<float>(p, a, p->rec);
    }
  }
  if (e == hipSuccess) {
    if (p->prec == ENUFFT_F64)
      hipLaunchKernelGGL(rec_finalize_kernel<double>, dim3((unsigned)p->n_cells), dim3(256), 0, p->stream,
                         (const double *)coef, keep, area, (const double *)p->d_rec_part,
                         (const int32_t *)p->d_cell_items, (const int64_t *)p->d_cell_item_off,
                         (const int64_t *)p->d_cell_off, p->geom, diag);
    else
      hipLaunchKernelGGL(rec_finalize_kernel<float>, dim3((unsigned)p->n_cells), dim3(256), 0, p->stream,
                         (const float *)coef, keep, area, (const double *)p->d_rec_part,
                         (const int32_t *)p->d_cell_items, (const int64_t *)p->d_cell_item_off,
                         (const int64_t *)p->d_cell_off, p->geom, diag);
    e = hipGetLastError();
  }
  if (e != hipSuccess) {
    p->last_error = std::string("enufft_reconstruct launch: ") + hipGetErrorString(e);
    p->faulted = true;
    return ENUFFT_EDEVICE;
  }
  return ENUFFT_OK;
}
