// FP64 large-cell spreading and gather on the matrix cores (included by big.hip after
// the tiled passes' arguments and work-unit loop).
//
// A point's W x W contributions are the outer product of its y and x taps, and its
// interpolation the two contractions of a grid window with them.  Points whose
// footprints start within BS x BS fine cells share one 16 x 16 window, so four of
// them are one v_mfma_f64_16x16x4 in the spreading (K runs over the points), and
// sixteen of them are twelve in the gather (the window's rows against the y taps
// of each point, for u, du/dx and du/dy; the x taps then weight the results).  Each
// unit's points are counted into the (32 / BS + 1)^2 such blocks of its tile in LDS.
//
// Why: one point per lane, a point is W^2 LDS adds of FP64 (8.7 cycles per 64 without
// conflicts; lanes at unrelated places conflict about fourfold), or 3 W^2 LDS reads.
// 1e7 clustered points, 512 x 512 modes, W = 12: spreading 1.54 ms (92 cycles of a CU
// per point) to 0.57 ms, gather 2.16 ms (133) to 0.89 ms.  The matrix instructions
// are 4 and 12 cycles of a CU per point; what is left is the points' own arithmetic
// (taps, window, coordinates: about 600 FP64 instructions per 64 points each) at the
// two waves per SIMD that the tap coefficients in registers leave.
//
// Widths 8 to 12: the window leaves an origin span of 17 - W cells, BS the power of
// two within it (8 at W = 8, else 4).  W = 14 and 16 would leave blocks of 2 and 1
// cells, mostly padding unless a cell holds tens of points; they keep the kernels
// of one point per lane, as do narrower kernels, sparse cells (m64_use) and plans without
// the tap polynomials.
#pragma once

typedef double mfma_d4 __attribute__((ext_vector_type(4)));

constexpr int M64_SPREAD_THREADS = 512;
constexpr int M64_GATHER_THREADS = 512;    // the window and the tap coefficients need more
constexpr int M64_PER = 16;                // points per thread of one round
constexpr int M64_TAPS = 17;               // LDS pitch of a point's 16 window taps

template <int W>
struct M64 {
  static constexpr int BS = W <= 8 ? 8 : 4;              // block side (origins)
  static constexpr int NB = (BIG_TS + 1) / BS + 1;       // blocks per axis (origins 0 .. BIG_TS + 1)
  static constexpr int S = BIG_TS + W + 1;               // sub-grid side
  static_assert(BS + W <= 17 && NB * NB <= 128, "one 16 x 16 window per block, two blocks per lane of the scan");
  // entries of the point list of NT threads' points with every block padded to PAD
  static constexpr int list(int nt, int pad) { return (nt * M64_PER + NB * NB * (pad - 1) + 63) / 64 * 64; }
  // doubles of a wave's own LDS: sixteen points' y and x window taps, and the tap
  // coordinates, strength and origins of the 64 points of a round
  static constexpr int wave_lds = 2 * 16 * M64_TAPS + 4 * 64;
};

__device__ __forceinline__ void m64_wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The points [k0, k1) of a tile (at most M64_PER per thread) listed by block: list[]
// holds their offsets from k0, 0xffff in the entries that pad each block to PAD.
// Returns the entries used.  The order inside a block is that of the LDS counters.
template <int W, int NT, int PAD>
__device__ int m64_list(const BigTileArgs<double> &a, const double *X, const double *Y, int64_t k0, int64_t k1, int tx0,
                        int ty0, int *cnt, uint16_t *list) {
  constexpr int NB = M64<W>::NB, BS = M64<W>::BS, NN = NB * NB, U = 4;
  const int t = threadIdx.x, n = (int)(k1 - k0);
  if (t < 128) cnt[t] = 0;
  for (int i = t; i < M64<W>::list(NT, PAD) / 2; i += NT) reinterpret_cast<unsigned *>(list)[i] = 0xffffffffu;
  __syncthreads();
  int at[M64_PER];   // block | place in it << 8
#pragma unroll
  for (int u0 = 0; u0 < M64_PER; u0 += U) {
    double xv[U], yv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t k = k0 + min(t + (u0 + u) * NT, n - 1);
      xv[u] = X[k];
      yv[u] = Y[k];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int lx = big_local(fine_coord<double>(xv[u], a.s1h, a.s1l, W * 0.5).i0 & (a.g.n1 - 1), tx0, a.g.n1);
      const int ly = big_local(fine_coord<double>(yv[u], a.s2h, a.s2l, W * 0.5).i0 & (a.g.n2 - 1), ty0, a.g.n2);
      const int b = (ly / BS) * NB + lx / BS;
      at[u0 + u] = t + (u0 + u) * NT < n ? b | atomicAdd(&cnt[b], 1) << 8 : -1;
    }
    if (u0 * NT + U * NT >= n) {   // the same in every thread
#pragma unroll
      for (int u = u0 + U; u < M64_PER; ++u) at[u] = -1;
      break;
    }
  }
  __syncthreads();
  if (t < 64) {   // counts become starts, each block's count rounded up to PAD
    const int c0 = 2 * t < NN ? (cnt[2 * t] + PAD - 1) / PAD * PAD : 0;
    const int c1 = 2 * t + 1 < NN ? (cnt[2 * t + 1] + PAD - 1) / PAD * PAD : 0;
    int inc = c0 + c1;
    for (int o = 1; o < 64; o <<= 1) {
      const int v = __shfl_up(inc, o, 64);
      if (t >= o) inc += v;
    }
    cnt[2 * t] = inc - c0 - c1;
    cnt[2 * t + 1] = inc - c1;
    if (t == 63) cnt[128] = inc;
  }
  __syncthreads();
  const int total = cnt[128];
#pragma unroll
  for (int u = 0; u < M64_PER; ++u)
    if (at[u] >= 0) list[cnt[at[u] & 0xff] + (at[u] >> 8)] = (uint16_t)(t + u * NT);
  __syncthreads();
  return total;
}

// Taps of sixteen points at a time: lane group lk = lane / 16 evaluates for point
// lane % 16 half of the mirror pairs of one axis (groups 0 and 1: y, 2 and 3: x), whose
// coefficients it keeps in registers, and writes them at the point's place in the
// block's window, with its half of the zeros beside them.
template <int W>
struct M64Taps {
  static constexpr int PP = (W / 2 + 1) / 2;   // pairs per lane (the second half may hold one fewer)
  double cf[PP][ES64_DEG + 1];
  int d0;                                      // first pair
  __device__ __forceinline__ void init(const EsPoly64 &es, int lk) {
    d0 = (lk & 1) * PP;
#pragma unroll
    for (int p = 0; p < PP; ++p)
#pragma unroll
      for (int k = 0; k <= ES64_DEG; ++k) cf[p][k] = es.c[min(d0 + p, W / 2 - 1) * (ES64_DEG + 1) + k];
  }
  // dst: the point's 16 window taps; o its origin in the window; c a factor
  __device__ __forceinline__ void put(double *dst, int o, double u, double c) const {
    // (an origin one cell past the block, should two evaluations of it differ, still
    // fits the window's span)
    o = min(max(o, 0), 16 - W);
    const double s = u * u;
#pragma unroll
    for (int p = 0; p < PP; ++p) {
      double e = cf[p][ES64_DEG - 1], q = cf[p][ES64_DEG];
#pragma unroll
      for (int k = ES64_DEG - 3; k >= 0; k -= 2) {
        e = fma(e, s, cf[p][k]);
        q = fma(q, s, cf[p][k + 1]);
      }
      if (2 * PP == W / 2 || p + 1 < PP || d0 == 0) {
        dst[o + d0 + p] = c * fma(u, q, e);
        dst[o + W - 1 - d0 - p] = c * fma(-u, q, e);
      }
    }
    const int z = o + W + (d0 ? (16 - W) / 2 : 0);
#pragma unroll
    for (int d = 0; d < (16 - W) / 2; ++d) dst[(z + d) & 15] = 0.0;
  }
};

template <int W>
__global__ __launch_bounds__(M64_SPREAD_THREADS) void big_spread64_kernel(BigTileArgs<double> a) {
  constexpr int S = M64<W>::S, BS = M64<W>::BS, NB = M64<W>::NB, NT = M64_SPREAD_THREADS, NWV = NT / 64;
  extern __shared__ __align__(16) unsigned char m64_raw[];
  double *sub = reinterpret_cast<double *>(m64_raw);
  double *taps = sub + S * S + (threadIdx.x >> 6) * M64<W>::wave_lds;   // this wave's: y, then x
  double *pts = taps + 2 * 16 * M64_TAPS;                               // (uy, ux, c, origins) by plane
  uint16_t *list = reinterpret_cast<uint16_t *>(sub + S * S + NWV * M64<W>::wave_lds);
  __shared__ int cnt[129];
  __shared__ int s_unit;
  const double *wn = a.windows + 3 * a.cell;
  const double cx = wn[0], cy = wn[1], R = wn[2];
  const double pr = R > 0.0 ? M_PI / R : 0.0;
  const bool pre = a.presorted[0];
  const double *X = pre ? a.xi : a.xs, *Y = pre ? a.yi : a.ys, *Hh = pre ? a.hi : a.hs, *Wq = pre ? a.wi : a.ws;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, li = lane & 15, lk = lane >> 4;
  M64Taps<W> tp;
  tp.init(a.es64, lk);
  big_units<double>(a, &s_unit, [&](int t, int64_t lo, int64_t hi, int u) {
    for (int i = threadIdx.x; i < S * S; i += NT) sub[i] = 0.0;
    const int tx0 = (t % a.ntx) * BIG_TS, ty0 = (t / a.ntx) * BIG_TS;
    for (int64_t k0 = lo; k0 < hi; k0 += NT * M64_PER) {
      const int64_t k1 = min(hi, k0 + NT * M64_PER);
      const int total = m64_list<W, NT, 4>(a, X, Y, k0, k1, tx0, ty0, cnt, list);
      // each wave takes consecutive rounds of 64 entries, so it rarely changes block
      const int rounds = (total + 63) / 64, per = (rounds + NWV - 1) / NWV;
      mfma_d4 acc = {0.0, 0.0, 0.0, 0.0};
      int block = -1;   // of acc (the same in every lane)
      auto flush = [&] {
        if (block < 0) return;
        const int r0 = (block / NB) * BS, c = (block % NB) * BS + li;
        if (c < S) {
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (r0 + 4 * r + lk < S)
              __hip_atomic_fetch_add(sub + (r0 + 4 * r + lk) * S + c, acc[r], __ATOMIC_RELAXED,
                                     __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        acc = mfma_d4{0.0, 0.0, 0.0, 0.0};
      };
      for (int q = wave * per; q < min(rounds, (wave + 1) * per); ++q) {
        const int e = q * 64 + lane < total ? (int)list[q * 64 + lane] : 0xffff;
        const bool on = e != 0xffff;
        const int64_t k = k0 + (on ? e : 0);
        const double xj = X[k], yj = Y[k];
        const double cj = on ? Wq[k] * Hh[k] * hann_w(a.window_kind, xj, yj, cx, cy, R, pr) : 0.0;
        const FineCoord<double> fx = fine_coord<double>(xj, a.s1h, a.s1l, W * 0.5);
        const FineCoord<double> fy = fine_coord<double>(yj, a.s2h, a.s2l, W * 0.5);
        const int lx = big_local(fx.i0 & (a.g.n1 - 1), tx0, a.g.n1);
        const int ly = big_local(fy.i0 & (a.g.n2 - 1), ty0, a.g.n2);
        // a group of four entries lies in one block, its first entry a point (or past
        // the list's end)
        const int bin = __shfl(on ? (ly / BS) * NB + lx / BS : -1, lane & ~3, 64);
        const int ox = lx - max(bin, 0) % NB * BS, oy = ly - max(bin, 0) / NB * BS;
        m64_wave_sync();
        pts[lane] = tap_u64(fy, W * 0.5);
        pts[64 + lane] = tap_u64(fx, W * 0.5);
        pts[128 + lane] = cj;
        reinterpret_cast<int2 *>(pts + 192)[lane] = make_int2(oy, ox);
        m64_wave_sync();
#pragma unroll 1
        for (int s = 0; s < 4; ++s) {   // sixteen points' taps at a time through LDS
          const int p = 16 * s + li, ax = lk >> 1;
          tp.put(taps + (16 * ax + li) * M64_TAPS, reinterpret_cast<const int *>(pts + 192)[2 * p + ax],
                 pts[64 * ax + p], ax ? 1.0 : pts[128 + p]);
          m64_wave_sync();
          double av[4], bv[4];
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            av[g] = taps[(4 * g + lk) * M64_TAPS + li];
            bv[g] = taps[(16 + 4 * g + lk) * M64_TAPS + li];
          }
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            const int b = __builtin_amdgcn_readlane(bin, 16 * s + 4 * g);
            if (b < 0) continue;
            if (b != block) {
              flush();
              block = b;
            }
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(av[g], bv[g], acc, 0, 0, 0);
          }
          m64_wave_sync();
        }
      }
      flush();
      __syncthreads();
    }
    double *dst = a.partial + (int64_t)u * (S * S);
    for (int i = threadIdx.x; i < S * S; i += NT) dst[i] = sub[i];
    __syncthreads();
  });
}

// Sum over the four lane groups of sixteen (every lane gets it): the halves' and then
// the neighbouring rows' values exchanged in registers.
__device__ __forceinline__ double m64_group_sum(double v) {
  const unsigned lo = (unsigned)__double2loint(v), hi = (unsigned)__double2hiint(v);
  const auto l32 = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
  const auto h32 = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
  v = __hiloint2double((int)h32[0], (int)l32[0]) + __hiloint2double((int)h32[1], (int)l32[1]);
  const unsigned lo2 = (unsigned)__double2loint(v), hi2 = (unsigned)__double2hiint(v);
  const auto l16 = __builtin_amdgcn_permlane16_swap(lo2, lo2, false, false);
  const auto h16 = __builtin_amdgcn_permlane16_swap(hi2, hi2, false, false);
  return __hiloint2double((int)h16[0], (int)l16[0]) + __hiloint2double((int)h16[1], (int)l16[1]);
}

template <int W>
__global__ __launch_bounds__(M64_GATHER_THREADS) void big_gather64_kernel(BigTileArgs<double> a) {
  constexpr int S = M64<W>::S, BS = M64<W>::BS, NB = M64<W>::NB, NT = M64_GATHER_THREADS, NWV = NT / 64;
  extern __shared__ __align__(16) unsigned char m64_raw[];
  double *su = reinterpret_cast<double *>(m64_raw);   // [3][S * S]: u, du/dx, du/dy
  double *taps = su + 3 * S * S + (threadIdx.x >> 6) * M64<W>::wave_lds;
  double *pts = taps + 2 * 16 * M64_TAPS;
  uint16_t *list = reinterpret_cast<uint16_t *>(su + 3 * S * S + NWV * M64<W>::wave_lds);
  __shared__ int cnt[129];
  __shared__ int s_unit;
  const Geom &g = a.g;
  const double *wn = a.windows + 3 * a.cell;
  const double cx = wn[0], cy = wn[1], R = wn[2];
  const double pr = R > 0.0 ? M_PI / R : 0.0;
  const bool pre = *a.presorted;
  const double *X = pre ? a.xi : a.xs, *Y = pre ? a.yi : a.ys, *Hh = pre ? a.hi : a.hs, *Wq = pre ? a.wi : a.ws;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, li = lane & 15, lk = lane >> 4;
  M64Taps<W> tp;
  tp.init(a.es64, lk);
  big_units<double>(a, &s_unit, [&](int t, int64_t lo, int64_t hi, int) {
    const int tx0 = (t % a.ntx) * BIG_TS, ty0 = (t / a.ntx) * BIG_TS;
    for (int i = threadIdx.x; i < S * S; i += NT) {
      const int r = i / S, q = i - r * S;
      const double4 v = a.G4[(int64_t)((ty0 - 1 + r) & (g.n2 - 1)) * g.n1 + ((tx0 - 1 + q) & (g.n1 - 1))];
      su[i] = v.x;
      su[S * S + i] = v.y;
      su[2 * S * S + i] = v.z;
    }
    for (int64_t k0 = lo; k0 < hi; k0 += NT * M64_PER) {
      const int64_t k1 = min(hi, k0 + NT * M64_PER);
      const int total = m64_list<W, NT, 16>(a, X, Y, k0, k1, tx0, ty0, cnt, list);
      const int rounds = (total + 63) / 64, per = (rounds + NWV - 1) / NWV;
      int block = -1;
      double wv[3][4];   // the block's window, transposed: columns by lane, rows 4 m + lk
#pragma unroll
      for (int m = 0; m < 12; ++m) wv[m / 4][m % 4] = 0.0;
      for (int q = wave * per; q < min(rounds, (wave + 1) * per); ++q) {
        const int e = q * 64 + lane < total ? (int)list[q * 64 + lane] : 0xffff;
        const bool on = e != 0xffff;
        const int64_t k = k0 + (on ? e : 0);
        const double xj = X[k], yj = Y[k], hj = Hh[k], wj = Wq[k];
        const FineCoord<double> fx = fine_coord<double>(xj, a.s1h, a.s1l, W * 0.5);
        const FineCoord<double> fy = fine_coord<double>(yj, a.s2h, a.s2l, W * 0.5);
        const int lx = big_local(fx.i0 & (g.n1 - 1), tx0, g.n1);
        const int ly = big_local(fy.i0 & (g.n2 - 1), ty0, g.n2);
        // sixteen entries lie in one block, their first a point (or past the list's end)
        const int bin = __shfl(on ? (ly / BS) * NB + lx / BS : -1, lane & ~15, 64);
        const int ox = lx - max(bin, 0) % NB * BS, oy = ly - max(bin, 0) / NB * BS;
        m64_wave_sync();
        pts[lane] = tap_u64(fy, W * 0.5);
        pts[64 + lane] = tap_u64(fx, W * 0.5);
        reinterpret_cast<int2 *>(pts + 192)[lane] = make_int2(oy, ox);
        m64_wave_sync();
        double val[3] = {0.0, 0.0, 0.0};
#pragma unroll 1
        for (int s = 0; s < 4; ++s) {
          const int b = __builtin_amdgcn_readlane(bin, 16 * s);
          if (b < 0) break;   // past the list's end
          const int p = 16 * s + li, ax = lk >> 1;
          tp.put(taps + (16 * ax + li) * M64_TAPS, reinterpret_cast<const int *>(pts + 192)[2 * p + ax],
                 pts[64 * ax + p], 1.0);
          m64_wave_sync();
          if (b != block) {
            block = b;
            // (cells past the sub-grid meet zero taps only; staged cells are read in
            // their place)
            const int r0 = (b / NB) * BS, c = min((b % NB) * BS + li, S - 1);
#pragma unroll
            for (int m = 0; m < 4; ++m) {
              const int at = min(r0 + 4 * m + lk, S - 1) * S + c;
              wv[0][m] = su[at];
              wv[1][m] = su[S * S + at];
              wv[2][m] = su[2 * S * S + at];
            }
          }
          double ty[4], tx[4];
#pragma unroll
          for (int m = 0; m < 4; ++m) {
            ty[m] = taps[li * M64_TAPS + 4 * m + lk];
            tx[m] = taps[(16 + li) * M64_TAPS + 4 * m + lk];
          }
          // acc[v][r]: column 4 r + lk of the window, contracted with point li's y taps
          mfma_d4 acc[3];
#pragma unroll
          for (int m = 0; m < 4; ++m)
#pragma unroll
            for (int v = 0; v < 3; ++v)
              acc[v] = __builtin_amdgcn_mfma_f64_16x16x4f64(wv[v][m], ty[m], m ? acc[v] : mfma_d4{0.0, 0.0, 0.0, 0.0},
                                                            0, 0, 0);
#pragma unroll
          for (int v = 0; v < 3; ++v) {
            double sum = acc[v][0] * tx[0];
#pragma unroll
            for (int r = 1; r < 4; ++r) sum = fma(acc[v][r], tx[r], sum);
            sum = m64_group_sum(sum);
            val[v] = lk == s ? sum : val[v];
          }
          m64_wave_sync();
        }
        if (on) {
          double dWx, dWy;
          const double Wv = hann_wg(a.window_kind, xj, yj, cx, cy, R, pr, dWx, dWy);
          const double wh = wj * hj;
          double4 o;
          o.x = wj * Wv * val[0];
          o.y = wh * (dWx * val[0] + Wv * val[1]);
          o.z = wh * (dWy * val[0] + Wv * val[2]);
          o.w = 0.0;
          if (pre) {   // the sorted position is the input position: the gradients go straight out
            if (a.gh) a.gh[k] = o.x;
            if (a.gx) a.gx[k] = o.y;
            if (a.gy) a.gy[k] = o.z;
          } else {
            a.gout[k] = o;
          }
        }
      }
      __syncthreads();
    }
  });
}

template <int W>
constexpr size_t m64_lds(bool gather) {
  constexpr size_t planes = M64<W>::S * M64<W>::S;
  const int nt = gather ? M64_GATHER_THREADS : M64_SPREAD_THREADS;
  return sizeof(double) * ((gather ? 3 * planes : planes) + (size_t)(nt / 64) * M64<W>::wave_lds) +
         sizeof(uint16_t) * M64<W>::list(nt, gather ? 16 : 4);
}

// Whether a cell's FP64 unit passes run on the matrix cores, and their launches.
//
// The blocks' padding, and a workgroup's list and its one place per CU, cost 4 (spreading)
// to 9 us (gather) per tile of a CU more than the kernels of one point per lane; what is
// won grows with the points that share a tile's cells.  Both forms, us (type-1, adjoint),
// W = 12, clustered points on 1,024 tiles: 35 points a tile 180 and 186, 211 and 217; 100
// 208 and 192, 281 and 232; 300 294 and 204, 441 and 290.  Even points lose until about 200
// to 400 a tile (100: 184 and 192, 216 and 244; 450: 216 and 213, 273 and 274).  On 4,096 tiles, where
// each CU takes sixteen, 100 clustered points 354 and 380, 532 and 563; 200 468 and 404,
// 727 and 646; even ones 381 and 406 at 200.  W = 8 and 10 lie close to this.  At W = 6 and
// below nothing is won (1e6 clustered points 323 and 315; 700 a tile 290 and 296, even 206 and 222).
constexpr double M64_PER_TILE = 96.0, M64_PER_TILE_MANY = 200.0;
inline bool m64_use(enufft_plan_t p, const EsPoly64 &es64, int64_t n) {
  return es64.on && p->W >= 8 && p->W <= 12 && (double)n >= p->m64_per_tile * p->big_ntx * p->big_nty;
}

template <int W>
hipError_t m64_launch_w(const BigTileArgs<double> &a, bool gather, int blocks, hipStream_t s) {
  const void *fn = gather ? (const void *)&big_gather64_kernel<W> : (const void *)&big_spread64_kernel<W>;
  void *args[] = {const_cast<BigTileArgs<double> *>(&a)};
  return hipLaunchKernel(fn, dim3(blocks), dim3(gather ? M64_GATHER_THREADS : M64_SPREAD_THREADS), args, m64_lds<W>(gather), s);
}

inline hipError_t m64_launch(int W, const BigTileArgs<double> &a, bool gather, int blocks, hipStream_t s) {
  switch (W) {
    case 8: return m64_launch_w<8>(a, gather, blocks, s);
    case 10: return m64_launch_w<10>(a, gather, blocks, s);
    case 12: return m64_launch_w<12>(a, gather, blocks, s);
    default: return hipErrorInvalidValue;
  }
}

template <int W>
hipError_t m64_attr_w() {
  hipError_t e = hipFuncSetAttribute((const void *)&big_spread64_kernel<W>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                     (int)m64_lds<W>(false));
  if (e != hipSuccess) return e;
  return hipFuncSetAttribute((const void *)&big_gather64_kernel<W>, hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)m64_lds<W>(true));
}
inline hipError_t m64_attrs() {
  hipError_t e = m64_attr_w<8>();
  if (e == hipSuccess) e = m64_attr_w<10>();
  if (e == hipSuccess) e = m64_attr_w<12>();
  return e;
}
