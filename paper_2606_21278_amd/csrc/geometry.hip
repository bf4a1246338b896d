// Per-cell geometry of a triangular mesh (enufft_cell_geometry): local frames
// and the square spectral box of Appendix A1, the square / triangle / circle
// support masks, uniform or raster-Voronoi quadrature weights (Appendix A2,
// eqs. uniform_weights, raster_grid .. voronoi_weights) and deplaning by the
// weighted cell mean (Appendix A6, eq. alps_deplaning).
//
// One workgroup per cell.  Phases, separated by workgroup barriers:
//   0  thread 0: centroid, rotation, rotated vertices, H and the mask area;
//   1  every sample: local and box coordinates, the mask flag; with Voronoi
//      weights also its bin in an nb x nb grid over the box (LDS counters) and
//      its slot in that bin;
//   2  exclusive scan of the bin counters (LDS);
//   3  inside samples scattered by bin into a workspace copy (u_x, u_y, index);
//   4  every raster cell centre inside the mask finds its nearest inside
//      sample by rings of bins around its own, sixteen lanes to a centre, leaving
//      out bins that cannot hold a sample as near and stopping once no farther
//      ring can; the sample's count is incremented;
//   5  weights, their FP64 sum and the weighted mean; deplaned heights.
//
// What bounds it: the longest cell.  With one thread per raster centre every
// distance waited for its own load, and where a third of a cell's samples stand
// close together a centre met thousands of them in its nine nearest bins, one
// after another (1,024 cells, 2e7 samples, 30 % of each cell's samples clustered,
// N_g = 64: 10.4 ms, nearly all of it the search in the largest cells).  A centre's
// own bin is searched first and bounds the rest, so a dense neighbourhood costs
// one or two bins; the samples of a row of bins are one contiguous range, which
// sixteen lanes read together.  With four samples per thread in flight and fewer
// passes over them (weights and mean in one): 10.86 to 1.87 ms a call.
// Decisions that yield integers (mask flags, nearest samples) use FP64 with
// contraction off, so they are exact functions of the FP64 inputs.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <string>
#include <vector>

#include "plan.h"

namespace enufft {
namespace {

constexpr int kGeoThreads = 1024;
constexpr int kGeoLanes = 16;                    // lanes that search for one raster centre
constexpr int kGeoUnroll = 4;                    // samples per thread and round, their loads issued together
constexpr int kGeoMaxBins = 128;                 // bins per axis
constexpr int kNoSample = 0x7fffffff;

struct GeoParams {
  int frame, mask, weights, raster, deplane;
  double eta, floor_frac;
};

struct GeoFrame {
  double cx, cy, cs, sn, H, area;
  double ut[6];                                   // rotated vertices
};

// Sutherland-Hodgman: the rotated triangle cut by the four half-planes of the
// box [-H, H]^2, then the shoelace area of what is left.
__device__ double tri_box_area(const double *ut, double H) {
#pragma clang fp contract(off)
  double ax[10], ay[10], bx[10], by[10];
  int n = 3;
  for (int i = 0; i < 3; ++i) { ax[i] = ut[2 * i]; ay[i] = ut[2 * i + 1]; }
  for (int side = 0; side < 4; ++side) {
    const bool on_y = side >= 2;
    const double s = (side & 1) ? -1.0 : 1.0;
    int m = 0;
    for (int i = 0; i < n; ++i) {
      const int k = (i + 1 == n) ? 0 : i + 1;
      const double pa = s * (on_y ? ay[i] : ax[i]) - H;
      const double pb = s * (on_y ? ay[k] : ax[k]) - H;
      if (pa <= 0.0) { bx[m] = ax[i]; by[m] = ay[i]; ++m; }
      if ((pa < 0.0 && pb > 0.0) || (pa > 0.0 && pb < 0.0)) {
        const double t = pa / (pa - pb);
        bx[m] = ax[i] + t * (ax[k] - ax[i]);
        by[m] = ay[i] + t * (ay[k] - ay[i]);
        ++m;
      }
    }
    n = m;
    for (int i = 0; i < n; ++i) { ax[i] = bx[i]; ay[i] = by[i]; }
  }
  double s2 = 0.0;
  for (int i = 0; i < n; ++i) {
    const int k = (i + 1 == n) ? 0 : i + 1;
    s2 += ax[i] * ay[k] - ax[k] * ay[i];
  }
  return 0.5 * fabs(s2);
}

// (Not inlined: one thread runs it per cell, and its clipping arrays would take the
// registers of the whole kernel.)
__device__ __noinline__ void make_frame(const double *v, const GeoParams &g, GeoFrame &F) {
#pragma clang fp contract(off)
  F.cx = (v[0] + v[2] + v[4]) / 3.0;
  F.cy = (v[1] + v[3] + v[5]) / 3.0;
  double cs = 1.0, sn = 0.0;
  if (g.frame == ENUFFT_FRAME_EDGE) {
    // edges v2 - v1, v3 - v2, v1 - v3; the first of the longest
    double best = -1.0, ex = 0.0, ey = 0.0;
    for (int i = 0; i < 3; ++i) {
      const int k = (i + 1) % 3;
      const double dx = v[2 * k] - v[2 * i], dy = v[2 * k + 1] - v[2 * i + 1];
      const double len = sqrt(dx * dx + dy * dy);
      if (len > best) { best = len; ex = dx; ey = dy; }
    }
    cs = ex / best;
    sn = ey / best;
  }
  F.cs = cs;
  F.sn = sn;
  double lo_x = 0.0, hi_x = 0.0, lo_y = 0.0, hi_y = 0.0;
  for (int i = 0; i < 3; ++i) {
    const double dx = v[2 * i] - F.cx, dy = v[2 * i + 1] - F.cy;
    const double ux = cs * dx + sn * dy, uy = -sn * dx + cs * dy;
    F.ut[2 * i] = ux;
    F.ut[2 * i + 1] = uy;
    lo_x = i ? fmin(lo_x, ux) : ux;
    hi_x = i ? fmax(hi_x, ux) : ux;
    lo_y = i ? fmin(lo_y, uy) : uy;
    hi_y = i ? fmax(hi_y, uy) : uy;
  }
  F.H = 0.5 * g.eta * fmax(hi_x - lo_x, hi_y - lo_y);
  if (g.mask == ENUFFT_MASK_SQUARE) F.area = 4.0 * F.H * F.H;
  else if (g.mask == ENUFFT_MASK_CIRCLE) F.area = M_PI * F.H * F.H;
  else F.area = tri_box_area(F.ut, F.H);
}

// Mask membership of a local point.  The triangle test takes the orientation
// of the point against each edge traversed v2 -> v1, v3 -> v2, v1 -> v3 (base
// at the edge's start); on the triangle when no two orientations have opposite
// signs.
__device__ bool in_support(const GeoFrame &F, int mask, double ux, double uy) {
#pragma clang fp contract(off)
  const double H = F.H;
  if (mask == ENUFFT_MASK_CIRCLE) return ux * ux + uy * uy <= H * H;
  if (!(fabs(ux) <= H && fabs(uy) <= H)) return false;
  if (mask == ENUFFT_MASK_SQUARE) return true;
  const double *t = F.ut;
  bool neg = false, pos = false;
  for (int e = 0; e < 3; ++e) {
    const int s = (e + 1) % 3, d = e;          // start vertex s, end vertex d
    const double o = (ux - t[2 * s]) * (t[2 * d + 1] - t[2 * s + 1]) - (t[2 * d] - t[2 * s]) * (uy - t[2 * s + 1]);
    neg = neg || (o < 0.0);
    pos = pos || (o > 0.0);
  }
  return !(neg && pos);
}

__device__ inline void to_local(const GeoFrame &F, double x, double y, double &ux, double &uy) {
#pragma clang fp contract(off)
  const double dx = x - F.cx, dy = y - F.cy;
  ux = F.cs * dx + F.sn * dy;
  uy = -F.sn * dx + F.cs * dy;
}

__device__ inline int bin_of(double u, double H, double inv_bw, int nb) {
  const int b = (int)floor((u + H) * inv_bw);
  return b < 0 ? 0 : (b >= nb ? nb - 1 : b);
}

// Workgroup sum of one double per thread (waves, then the wave sums; fixed order).
__device__ double wg_sum(double v, double *red) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  double s = 0.0;
  for (int w = 0; w < kGeoThreads / 64; ++w) s += red[w];
  return s;
}

// Nearest inside sample of the raster centre (gx, gy), found by the kGeoLanes lanes
// of a group together; every lane returns its index in the cell (ties to the lowest;
// kNoSample only where no distance is a number).
// u, id: the samples in bin order; bins: the bins' first positions.
__device__ int nearest_sample(double gx, double gy, double H, double bw, double inv_bw, int nb, const int *bins,
                              const double2 *__restrict__ u, const int32_t *__restrict__ id) {
#pragma clang fp contract(off)
  const int gl = threadIdx.x & (kGeoLanes - 1);
  const int bx = bin_of(gx, H, inv_bw, nb), by = bin_of(gy, H, inv_bw, nb);
  const double slack = 1e-9 * bw;   // covers the rounding of the bin index
  const double far = __builtin_inf();
  double bd = far, gd = far;        // best squared distance: this lane's, the group's
  int arg = -1;                     // its position
  auto scan = [&](int p0, int p1) {
    for (int p = p0 + gl; p < p1; p += 2 * kGeoLanes) {
      const int q = p + kGeoLanes < p1 ? p + kGeoLanes : p;
      const double2 v0 = u[p], v1 = u[q];
      const double d0 = (v0.x - gx) * (v0.x - gx) + (v0.y - gy) * (v0.y - gy);
      const double d1 = (v1.x - gx) * (v1.x - gx) + (v1.y - gy) * (v1.y - gy);
      if (d0 < bd || (d0 == bd && (arg < 0 || id[p] < id[arg]))) { bd = d0; arg = p; }
      if (q != p && (d1 < bd || (d1 == bd && (arg < 0 || id[q] < id[arg])))) { bd = d1; arg = q; }
    }
  };
  auto share = [&] {
    gd = bd;
    for (int o = 1; o < kGeoLanes; o <<= 1) gd = fmin(gd, __shfl_xor(gd, o, 64));
  };
  // lower bound of the distance along one axis from g to bin k of that axis
  auto gap = [&](double g, int gbin, int k) {
    const double e = k > gbin ? (-H + bw * k) - g - slack : k < gbin ? g - (-H + bw * (k + 1)) - slack : 0.0;
    return e > 0.0 ? e : 0.0;
  };
  for (int ring = 0; ring < nb; ++ring) {
    const int y0 = by - ring, y1 = by + ring;
    for (int yy = y0 > 0 ? y0 : 0; yy <= y1 && yy < nb; ++yy) {
      const double dy = gap(gy, by, yy), dy2 = dy * dy;
      if (dy2 > gd) continue;
      const int *row = bins + yy * nb;
      if (yy == y0 || yy == y1) {
        int x0 = bx - ring > 0 ? bx - ring : 0, x1 = bx + ring < nb - 1 ? bx + ring : nb - 1;
        while (x0 < bx) {
          const double dx = gap(gx, bx, x0);
          if (dx * dx + dy2 <= gd) break;
          ++x0;
        }
        while (x1 > bx) {
          const double dx = gap(gx, bx, x1);
          if (dx * dx + dy2 <= gd) break;
          --x1;
        }
        scan(row[x0], row[x1 + 1]);
      } else {
        for (int side = 0; side < 2; ++side) {
          const int xx = side ? bx + ring : bx - ring;
          if (xx < 0 || xx >= nb) continue;
          const double dx = gap(gx, bx, xx);
          if (dx * dx + dy2 <= gd) scan(row[xx], row[xx + 1]);
        }
      }
      share();
    }
    // every bin beyond this ring is more than ring * bw away
    const double lim = (double)ring * bw * (1.0 - 1e-9);
    if (gd < lim * lim) break;
  }
  int who = arg >= 0 ? id[arg] : kNoSample;
  for (int o = 1; o < kGeoLanes; o <<= 1) {
    const double od = __shfl_xor(bd, o, 64);
    const int ow = __shfl_xor(who, o, 64);
    if (od < bd || (od == bd && ow < who)) { bd = od; who = ow; }
  }
  return who;
}

// Persistent workgroups take cells from a counter, largest cells first (the order
// array), so the largest cells do not end the launch alone; each workgroup keeps
// its Voronoi workspace in its own slice (the size of the largest cell).
template <typename T>
__global__ void __launch_bounds__(kGeoThreads) geometry_kernel(
    GeoParams g, const int32_t *__restrict__ order, int64_t n_cells, int *counter, int *done, int64_t slice,
    const int64_t *__restrict__ off, const double *__restrict__ tri,
    const T *__restrict__ x, const T *__restrict__ y, const T *__restrict__ h, T *__restrict__ xb,
    T *__restrict__ yb, T *__restrict__ hb, T *__restrict__ wb, uint8_t *__restrict__ inside,
    double *__restrict__ info, int32_t *__restrict__ counts, double2 *__restrict__ ws_u,
    int32_t *__restrict__ ws_idx, int32_t *__restrict__ ws_slot) {
#pragma clang fp contract(off)
  extern __shared__ __align__(16) unsigned char geo_lds[];
  __shared__ GeoFrame F;
  __shared__ double red[kGeoThreads / 64];
  __shared__ int part[kGeoThreads / 64];
  __shared__ int list[kGeoThreads];               // raster centres of a round inside the mask
  __shared__ int qin_s, nlist_s, s_idx;
  int *bins = reinterpret_cast<int *>(geo_lds);   // [nb * nb + 1] (Voronoi only)

  const int t = threadIdx.x;
  const int64_t base = (int64_t)blockIdx.x * slice;   // this workgroup's workspace slice
  for (;;) {
  if (t == 0) s_idx = atomicAdd(counter, 1);
  __syncthreads();
  const int64_t idx = s_idx;
  __syncthreads();
  if (idx >= n_cells) break;
  const int64_t c = order[idx];
  const int64_t a = off[c], b = off[c + 1];
  const int64_t Q = b - a;
  const bool vor = g.weights == ENUFFT_WEIGHTS_VORONOI;
  const int nb = vor ? (int)min<int64_t>(kGeoMaxBins, max<int64_t>(1, (int64_t)sqrt((double)Q / 3.0))) : 1;
  const int nbin = nb * nb;

  if (t == 0) {
    make_frame(tri + 6 * c, g, F);
    qin_s = 0;
    nlist_s = 0;
  }
  if (vor)
    for (int i = t; i <= nbin; i += kGeoThreads) bins[i] = 0;
  __syncthreads();
  const double H = F.H;
  const double inv_bw = (double)nb / (2.0 * H);

  // The loops over samples take kGeoUnroll per thread and round, loads first (past
  // the end: the last sample again, unused).
  constexpr int U = kGeoUnroll;
  const int64_t stride = (int64_t)U * kGeoThreads;

  // phase 1: coordinates, mask flags, bin slots (-1 outside the mask)
  int my_in = 0;
  for (int64_t j0 = a + t; j0 < b; j0 += stride) {
    T xv[U], yv[U];
#pragma unroll
    for (int q = 0; q < U; ++q) {
      const int64_t j = min(j0 + q * kGeoThreads, b - 1);
      xv[q] = x[j];
      yv[q] = y[j];
    }
#pragma unroll
    for (int q = 0; q < U; ++q) {
      const int64_t j = j0 + q * kGeoThreads;
      if (j >= b) break;
      double ux, uy;
      to_local(F, (double)xv[q], (double)yv[q], ux, uy);
      const bool in = in_support(F, g.mask, ux, uy);
      xb[j] = (T)(ux * M_PI / H);
      yb[j] = (T)(uy * M_PI / H);
      if (inside) inside[j] = in ? 1 : 0;
      if (counts) counts[j] = 0;
      my_in += in ? 1 : 0;
      if (vor) {
        const int bi = bin_of(uy, H, inv_bw, nb) * nb + bin_of(ux, H, inv_bw, nb);
        ws_slot[base + (j - a)] = in ? atomicAdd(&bins[bi], 1) : -1;
      }
    }
  }
  if (my_in) atomicAdd(&qin_s, my_in);
  __syncthreads();
  const int64_t qin = qin_s;

  double my_h = 0.0;
  if (vor && qin > 0) {
    // phase 2: exclusive scan of the bin counters
    const int per = (nbin + kGeoThreads - 1) / kGeoThreads;
    const int lo = min(nbin, t * per), hi = min(nbin, lo + per);
    int s = 0;
    for (int i = lo; i < hi; ++i) s += bins[i];
    int inc = s;
    for (int o = 1; o < 64; o <<= 1) {
      const int v = __shfl_up(inc, o, 64);
      if ((t & 63) >= o) inc += v;
    }
    if ((t & 63) == 63) part[t >> 6] = inc;
    __syncthreads();
    int run = inc - s;
    for (int w = 0; w < (t >> 6); ++w) run += part[w];
    for (int i = lo; i < hi; ++i) {
      const int cnt = bins[i];
      bins[i] = run;
      run += cnt;
    }
    if (t == kGeoThreads - 1) bins[nbin] = run;
    __syncthreads();

    // phase 3: scatter the inside samples by bin.  From here on ws_slot is the
    // count of each sample when the caller takes no counts: 0, or -1 outside the
    // mask (with counts it keeps the slots, -1 outside).
    int32_t *flag = ws_slot + base;
    for (int64_t j0 = a + t; j0 < b; j0 += stride) {
      T xv[U], yv[U];
      int sl[U];
#pragma unroll
      for (int q = 0; q < U; ++q) {
        const int64_t j = min(j0 + q * kGeoThreads, b - 1);
        xv[q] = x[j];
        yv[q] = y[j];
        sl[q] = flag[j - a];
      }
#pragma unroll
      for (int q = 0; q < U; ++q) {
        const int64_t j = j0 + q * kGeoThreads;
        if (j >= b || sl[q] < 0) continue;
        double ux, uy;
        to_local(F, (double)xv[q], (double)yv[q], ux, uy);
        const int bi = bin_of(uy, H, inv_bw, nb) * nb + bin_of(ux, H, inv_bw, nb);
        const int64_t pos = base + bins[bi] + sl[q];
        ws_u[pos] = make_double2(ux, uy);
        ws_idx[pos] = (int32_t)(j - a);
        if (!counts) flag[j - a] = 0;
      }
    }
    __syncthreads();

    // phase 4: nearest inside sample of every raster cell centre in the mask.  Each
    // round lists the centres of kGeoThreads raster points that are inside; groups
    // of lanes take them in turn.
    int32_t *cnt = counts ? counts + a : flag;
    const int Ng = g.raster;
    const double step = 2.0 * H / Ng;
    const double bw = 2.0 * H / nb;
    int64_t ng = 0;
    for (int64_t r0 = 0; r0 < (int64_t)Ng * Ng; r0 += kGeoThreads) {
      const int64_t r = r0 + t;
      if (r < (int64_t)Ng * Ng) {
        const double gx = -H + step * ((int)(r % Ng) + 0.5), gy = -H + step * ((int)(r / Ng) + 0.5);
        if (in_support(F, g.mask, gx, gy)) list[atomicAdd(&nlist_s, 1)] = (int)r;
      }
      __syncthreads();
      const int nl = nlist_s;
      ng += nl;
      for (int i = t / kGeoLanes; i < nl; i += kGeoThreads / kGeoLanes) {
        const int rr = list[i];
        const double gx = -H + step * (rr % Ng + 0.5), gy = -H + step * (rr / Ng + 0.5);
        const int who = nearest_sample(gx, gy, H, bw, inv_bw, nb, bins, ws_u + base, ws_idx + base);
        if ((t & (kGeoLanes - 1)) == 0 && who != kNoSample) atomicAdd(&cnt[who], 1);
      }
      __syncthreads();
      if (t == 0) nlist_s = 0;
      __syncthreads();
    }

    // phase 5: areas, their sum, the normalised weights and the weighted mean
    auto area = [&](int n, bool in) {
      return in && ng > 0 ? F.area * (n > 0 ? (double)n : g.floor_frac) / (double)ng : 0.0;
    };
    double my_tot = 0.0;
    for (int64_t j0 = t; j0 < Q; j0 += stride) {
      int n[U], fl[U];
#pragma unroll
      for (int q = 0; q < U; ++q) {
        const int64_t j = min(j0 + q * kGeoThreads, Q - 1);
        n[q] = cnt[j];
        fl[q] = flag[j];
      }
#pragma unroll
      for (int q = 0; q < U; ++q)
        if (j0 + q * kGeoThreads < Q) my_tot += area(n[q], fl[q] >= 0);
    }
    const double tot = wg_sum(my_tot, red);
    for (int64_t j0 = t; j0 < Q; j0 += stride) {
      int n[U], fl[U];
      T hv[U];
#pragma unroll
      for (int q = 0; q < U; ++q) {
        const int64_t j = min(j0 + q * kGeoThreads, Q - 1);
        n[q] = cnt[j];
        fl[q] = flag[j];
        hv[q] = h[a + j];
      }
#pragma unroll
      for (int q = 0; q < U; ++q) {
        const int64_t j = j0 + q * kGeoThreads;
        if (j >= Q) break;
        const double wq = tot > 0.0 ? area(n[q], fl[q] >= 0) / tot : 0.0;
        wb[a + j] = (T)wq;
        my_h += wq * (double)hv[q];
      }
    }
  } else {
    for (int64_t j0 = a + t; j0 < b; j0 += stride) {
      T xv[U], yv[U], hv[U];
#pragma unroll
      for (int q = 0; q < U; ++q) {
        const int64_t j = min(j0 + q * kGeoThreads, b - 1);
        xv[q] = x[j];
        yv[q] = y[j];
        hv[q] = h[j];
      }
#pragma unroll
      for (int q = 0; q < U; ++q) {
        const int64_t j = j0 + q * kGeoThreads;
        if (j >= b) break;
        double ux, uy;
        to_local(F, (double)xv[q], (double)yv[q], ux, uy);
        const bool in = in_support(F, g.mask, ux, uy);
        const double wq = (!vor && in) ? 1.0 / (double)qin : 0.0;
        wb[j] = (T)wq;
        my_h += wq * (double)hv[q];
      }
    }
  }

  // phase 6: the weighted mean and deplaning
  const double hbar = wg_sum(my_h, red);
  for (int64_t j0 = a + t; j0 < b; j0 += stride) {
    T hv[U];
#pragma unroll
    for (int q = 0; q < U; ++q) hv[q] = h[min(j0 + q * kGeoThreads, b - 1)];
#pragma unroll
    for (int q = 0; q < U; ++q) {
      const int64_t j = j0 + q * kGeoThreads;
      if (j < b) hb[j] = (T)(g.deplane ? (double)hv[q] - hbar : (double)hv[q]);
    }
  }
  if (t == 0 && info) {
    double *ci = info + 8 * c;
    ci[0] = F.cx; ci[1] = F.cy; ci[2] = F.cs; ci[3] = F.sn;
    ci[4] = F.H; ci[5] = F.area; ci[6] = (double)qin; ci[7] = g.deplane ? hbar : 0.0;
  }
  __syncthreads();   // the frame, bins and sums are the next cell's
  }
  if (t == 0) {
    __threadfence();
    if (atomicAdd(done, 1) == (int)gridDim.x - 1) {   // the last workgroup resets the counters
      *counter = 0;
      *done = 0;
    }
  }
}

}  // namespace
}  // namespace enufft

namespace enufft {
namespace {

// Bins per axis of a cell of Q samples (the kernel's rule).
int geo_bins(int64_t Q) {
  return (int)std::min<int64_t>(kGeoMaxBins, std::max<int64_t>(1, (int64_t)std::sqrt((double)Q / 3.0)));
}

// Workspace allocation recorded in the plan (released with the plan or by dev_release).
enufft_status geo_alloc(enufft_plan_t p, void **d, size_t bytes, const char *what) {
  hipError_t e = hipMalloc(d, std::max<size_t>(16, bytes));
  if (e != hipSuccess) {
    *d = nullptr;
    p->last_error = std::string("enufft_cell_geometry: ") + what + " allocation failed";
    return ENUFFT_ENOMEM;
  }
  p->allocations.push_back(*d);
  p->workspace_bytes += (int64_t)std::max<size_t>(16, bytes);
  return ENUFFT_OK;
}

enufft_status geo_fail(enufft_plan_t p, enufft_status st, const std::string &msg) {
  p->last_error = "enufft_cell_geometry: " + msg;
  return st;
}

template <typename T>
hipError_t geo_launch(enufft_plan_t p, const GeoParams &g, const int32_t *order, int blocks, int64_t slice, size_t lds, const double *tri,
                      const void *x, const void *y, const void *h, void *xb, void *yb, void *hb, void *wb,
                      uint8_t *inside, double *info, int32_t *counts, double2 *ws_u, int32_t *ws_idx,
                      int32_t *ws_slot) {
  auto fn = geometry_kernel<T>;
  hipLaunchKernelGGL(fn, dim3((unsigned)blocks), dim3(kGeoThreads), lds, p->stream, g, order,
                     p->n_cells, p->d_counters + 6, p->d_counters + 7, slice, (const int64_t *)p->d_cell_off, tri,
                     (const T *)x, (const T *)y, (const T *)h, (T *)xb, (T *)yb, (T *)hb, (T *)wb, inside, info,
                     counts, ws_u, ws_idx, ws_slot);
  return hipGetLastError();
}

template <typename T>
hipError_t geo_occupancy(size_t lds, int *per_cu) {
  hipError_t e = hipFuncSetAttribute((const void *)geometry_kernel<T>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                     (int)lds);
  if (e != hipSuccess) return e;
  return hipOccupancyMaxActiveBlocksPerMultiprocessor(per_cu, (const void *)geometry_kernel<T>, kGeoThreads, lds);
}

}  // namespace

enufft_status cell_offsets(enufft_plan_t p);
enufft_status geometry_supported(enufft_plan_t p);

}  // namespace enufft

extern "C" enufft_status enufft_cell_geometry(enufft_plan_t p, const double *tri, const void *x, const void *y,
                                              const void *h, const enufft_geometry_opts *opts, void *xb, void *yb,
                                              void *hb, void *wb, uint8_t *inside, double *info,
                                              int32_t *counts) {
  using namespace enufft;
  enufft_status st = check_plan(p, "enufft_cell_geometry");
  if (st != ENUFFT_OK) return st;
  if (!opts) return geo_fail(p, ENUFFT_EINVAL, "null options");
  const enufft_geometry_opts &o = *opts;
  if (o.frame < 0 || o.frame > 1 || o.mask < 0 || o.mask > 2 || o.weights < 0 || o.weights > 1)
    return geo_fail(p, ENUFFT_EINVAL, "unknown frame, mask or weights kind");
  if (!(o.eta >= 1.0) || !std::isfinite(o.eta) || !(o.floor_frac >= 0.0) || !std::isfinite(o.floor_frac))
    return geo_fail(p, ENUFFT_EINVAL, "eta must be finite and >= 1, floor_frac finite and >= 0");
  if (o.weights == ENUFFT_WEIGHTS_VORONOI && (o.raster < 1 || o.raster > 4096))
    return geo_fail(p, ENUFFT_EINVAL, "raster must be in [1, 4096] for Voronoi weights");
  if (p->n_cells == 0) return ENUFFT_OK;
  if (!tri) return geo_fail(p, ENUFFT_EINVAL, "null triangle array");
  if (p->n_points > 0 && (!x || !y || !h || !xb || !yb || !hb || !wb))
    return geo_fail(p, ENUFFT_EINVAL, "null point or output array");
  st = geometry_supported(p);
  if (st == ENUFFT_OK) st = cell_offsets(p);
  if (st != ENUFFT_OK) return st;
  const bool vor = o.weights == ENUFFT_WEIGHTS_VORONOI;
  GeoParams g{o.frame, o.mask, o.weights, o.raster, o.deplane ? 1 : 0, o.eta, o.floor_frac};

  // cells largest first (computed once per plan)
  int64_t largest = 0;
  for (int64_t c = 0; c < p->n_cells; ++c) largest = std::max(largest, p->offsets[c + 1] - p->offsets[c]);
  if (largest >= (int64_t(1) << 31)) return geo_fail(p, ENUFFT_EUNSUPPORTED, "cells of 2^31 points or more");
  const int32_t *order = nullptr;
  st = cells_largest_first(p, &order);
  if (st != ENUFFT_OK) return st;
  // persistent workgroups: as many as are resident (the Voronoi bins take the LDS
  // of the largest cell's bin grid)
  const int nbl = vor ? std::min(kGeoMaxBins, geo_bins(largest) + 1) : 0;
  const size_t lds = vor ? (size_t)(nbl * nbl + 1) * sizeof(int) : 16;
  int per_cu = 0;
  hipError_t e = p->prec == ENUFFT_F64 ? geo_occupancy<double>(lds, &per_cu) : geo_occupancy<float>(lds, &per_cu);
  if (e != hipSuccess || per_cu < 1) return geo_fail(p, ENUFFT_EDEVICE, "geometry kernel cannot be resident");
  const int blocks = (int)std::min<int64_t>(p->n_cells, (int64_t)p->n_cu * per_cu);
  const int64_t slice = vor ? largest : 0;
  const int64_t need = (int64_t)blocks * slice;
  if (vor && need > p->geo_ws_points) {
    dev_release(p, &p->geo_ws, (size_t)p->geo_ws_points * 16);
    dev_release(p, &p->geo_ws_i, (size_t)p->geo_ws_points * 8);
    p->geo_ws_points = 0;
    st = geo_alloc(p, &p->geo_ws, (size_t)std::max<int64_t>(1, need) * 16, "geometry sample copy");
    if (st == ENUFFT_OK)
      st = geo_alloc(p, &p->geo_ws_i, (size_t)std::max<int64_t>(1, need) * 8, "geometry sample index");
    if (st != ENUFFT_OK) return st;
    p->geo_ws_points = need;
  }
  double2 *ws_u = vor ? (double2 *)p->geo_ws : nullptr;
  int32_t *ws_idx = vor ? (int32_t *)p->geo_ws_i : nullptr;
  int32_t *ws_slot = vor ? ws_idx + p->geo_ws_points : nullptr;
  if (p->prec == ENUFFT_F64)
    e = geo_launch<double>(p, g, order, blocks, slice, lds, tri, x, y, h, xb, yb, hb, wb, inside, info, counts, ws_u, ws_idx,
                           ws_slot);
  else
    e = geo_launch<float>(p, g, order, blocks, slice, lds, tri, x, y, h, xb, yb, hb, wb, inside, info, counts, ws_u, ws_idx,
                          ws_slot);
  if (e != hipSuccess) {
    p->last_error = std::string("enufft_cell_geometry launch: ") + hipGetErrorString(e);
    p->faulted = true;
    return ENUFFT_EDEVICE;
  }
  return ENUFFT_OK;
}
