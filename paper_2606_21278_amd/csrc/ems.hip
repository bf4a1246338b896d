// Elastic Mode Selection on gfx950: one workgroup per cell; the unit energies stay in
// registers and their values are placed in LDS by bucket and rank (cells whose buckets
// crowd, or with negative energies: a comparison network per wave, merged through LDS).
//
// Section 2.2 of the paper, in its order: unit energies (eq. energy, with the
// optional weight of eq. weighted_e), the descending order of eq.
// sorted_energy, the participation ratio (eq. n_eff), the gap-ratio score
// (eq. s_delta), the combined measure and target fraction (eqs. c_score,
// alpha_c), the retained fraction (eq. f_cum) and the elastic count
// (eq. k_elastic).  Energies, sums, the running sum and the threshold test are
// FP64 so the ordering and the cut do not depend on FP32 rounding of the sums.
#include <algorithm>
#include <climits>
#include <cmath>
#include <cstdlib>
#include <string>
#include <vector>

#include "device_common.h"
#include "launch.h"
#include "plan.h"

namespace enufft {

struct EmsArgs {
  const void *f;
  const double *mode_weight;
  const double *flow;         // flow mode: [n_steps * n_cells_f][6] records (ux, uy, N, fc, rho, kscale)
  int64_t n_cells_f;          // flow mode: cells per step (the coefficients of cell v mod n_cells_f)
  uint8_t *keep;
  int32_t *k_star;
  double *stats;
  const int2 *units;          // (rep, partner | -1), ascending unit id
  int J;
  int M;                      // modes per cell = N1 * N2
  int N1, N2;                 // mode box (row-major, N1 modes per row)
  int64_t cell_begin, cell_end;
  int dc;                     // index of the excluded k = 0 mode, or -1
  int k_min, k_max;
  double alpha_min, alpha_max, delta, w1, w2;
};

// One wave per cell.  Wave-wide helpers: every lane returns the same value.
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ int wave_sum_i(int v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ int wave_min_i(int v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = min(v, __shfl_xor(v, o, 64));
  return v;
}
// Exclusive prefix over lanes (Hillis-Steele on the wave).
template <typename V>
__device__ __forceinline__ V wave_exclusive_scan(V v, int lane) {
  V inc = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const V t = __shfl_up(inc, o, 64);
    if (lane >= o) inc += t;
  }
  return inc - v;
}

// max / min of two energies.  The values are finite and never signalling
// NaNs, so the plain instructions do (the generic fmax would first quiet both
// operands).
__device__ __forceinline__ double dmax(double a, double b) {
  double r;
  asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
__device__ __forceinline__ double dmin(double a, double b) {
  double r;
  asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}

// Descending bitonic sort of the wave's JP = 64 R values held blocked (lane l
// holds positions l R .. l R + R - 1), in the flip form: for each block size
// k a flip comparator (i against i ^ (k - 1)) then half-cleaners j = k/4 .. 1;
// the lower index of every pair takes the larger value, so no direction bits.
// Pairs inside a lane are register compare-exchanges; pairs across lanes
// exchange through cross-lane shuffles.  Stages are template-expanded so every
// register index is a constant.
template <int R, int K>
__device__ __forceinline__ void flip_stage(double (&e)[R], int lane) {
  if constexpr (K <= R) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int q = r ^ (K - 1);
      if (r < q) {
        const double hi = dmax(e[r], e[q]), lo = dmin(e[r], e[q]);
        e[r] = hi; e[q] = lo;
      }
    }
  } else {
    constexpr int lm = K / R - 1;
    const bool lower = (lane & (K / (2 * R))) == 0;
#pragma unroll
    for (int r = 0; r < (R + 1) / 2; ++r) {
      const int q = R - 1 - r;
      const double o1 = __shfl_xor(e[q], lm, 64);   // partner of my r is the partner lane's q
      if (q != r) {
        const double o2 = __shfl_xor(e[r], lm, 64);
        const double h2 = dmax(e[q], o2), l2 = dmin(e[q], o2);
        e[q] = lower ? h2 : l2;
      }
      const double h1 = dmax(e[r], o1), l1 = dmin(e[r], o1);
      e[r] = lower ? h1 : l1;
      if ((r & 7) == 7) __builtin_amdgcn_sched_barrier(0);   // bound the shuffles in flight
    }
  }
}

template <int R, int J>
__device__ __forceinline__ void half_stages(double (&e)[R], int lane) {
  if constexpr (J >= 1) {
    if constexpr (J < R) {
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const int q = r ^ J;
        if (r < q) {
          const double hi = dmax(e[r], e[q]), lo = dmin(e[r], e[q]);
          e[r] = hi; e[q] = lo;
        }
      }
    } else {
      constexpr int lm = J / R;
      const bool lower = (lane & lm) == 0;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const double o = __shfl_xor(e[r], lm, 64);
        const double hi = dmax(e[r], o), lo = dmin(e[r], o);
        e[r] = lower ? hi : lo;
        if ((r & 15) == 15) __builtin_amdgcn_sched_barrier(0);
      }
    }
    half_stages<R, J / 2>(e, lane);
  }
}

template <int R, int K = 2>
__device__ __forceinline__ void wave_sort_desc(double (&e)[R], int lane) {
  if constexpr (K <= 64 * R) {
    flip_stage<R, K>(e, lane);
    half_stages<R, K / 4>(e, lane);
    wave_sort_desc<R, 2 * K>(e, lane);
  }
}

// Energy of unit u (FP64; products of FP32 values are exact in FP64) from its
// loaded coefficients and mode weights (1 without weights: the product by 1
// is exact).  Loads are unconditional (a missing partner reads the
// representative and is masked).  Every product and sum is rounded on its own
// (contraction into fused multiply-adds is off here), as the large cells' passes do.
__device__ __forceinline__ double member_energy(double re, double im, double w) {
#pragma clang fp contract(off)
  return (re * re + im * im) * w;
}

template <typename C>
__device__ __forceinline__ double pair_energy_v(const C fr, const C fp, double wr, double wp, bool partner) {
#pragma clang fp contract(off)
  const double e = member_energy((double)fr.x, (double)fr.y, wr);
  const double ep = member_energy((double)fp.x, (double)fp.y, wp);
  return partner ? e + ep : e;
}

// Flow mode: the weight of eq. (weighted_e) is the launch weight of an
// orographic gravity wave (Appendix A7) under the cell's flow record, in the
// paper's order: intrinsic frequency omega = -k . u (eq. mountain_omega), the
// vertical wave number from the dispersion relation (eq. mw_dispersion), the
// wave action of eq. (mw_action) per unit modal power, taken in magnitude (the
// action and omega share their signed branch, so the wave energy is positive).
// Modes outside the propagating band fc < |omega| < N, and k = 0, weigh 0.
// k = kscale (kx, ky) is the physical wave vector.
struct FlowRec {
  double ux, uy, N, fc, rho, ks;
  bool on;
};

__device__ __forceinline__ double flow_weight(const FlowRec &fl, int kx, int ky) {
#pragma clang fp contract(off)
  const double k1 = fl.ks * (double)kx, k2 = fl.ks * (double)ky;
  const double kk = k1 * k1 + k2 * k2;
  if (!(kk > 0.0)) return 0.0;
  const double omega = -(k1 * fl.ux + k2 * fl.uy);
  const double aw = fabs(omega);
  if (!(aw > fabs(fl.fc) && aw < fl.N)) return 0.0;
  const double m2 = kk * (fl.N * fl.N - omega * omega) / (omega * omega - fl.fc * fl.fc);
  const double act = -(fl.rho / 2.0) * (k1 * fl.ux + k2 * fl.uy) * (kk + m2) / kk;
  return fabs(act);
}

// Row of mode m (row-major, N1 per row; the float quotient is within one of the
// true one for the at most 2^13 modes of these kernels).
__device__ __forceinline__ int mode_row(int m, int N1, float inv_n1) {
  int r = (int)((float)m * inv_n1);
  r -= r * N1 > m;
  r += (r + 1) * N1 <= m;
  return r;
}

// The energies of n units with all loads of the batch issued before any is used:
// member indices first, then coefficients, then (with mode weights) the weights.
// reps[i] < 0 marks an entry with no unit (its energy is returned as 0).  The flow
// weight is the same for k and -k, bit for bit (the wave vector enters squared, or in
// one product whose magnitude is taken), so a pair's is evaluated once.
template <typename C, int N>
__device__ __forceinline__ void batch_energy(const EmsArgs &a, const FlowRec &fl, const C *f, const int (&reps)[N],
                                             const int (&partners)[N], double (&e)[N]) {
  C fr[N], fp[N];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const int rep = reps[i] >= 0 ? reps[i] : 0;
    fr[i] = f[rep];
    fp[i] = f[partners[i] >= 0 ? partners[i] : rep];
  }
  double wr[N], wp[N];
#pragma unroll
  for (int i = 0; i < N; ++i) wr[i] = wp[i] = 1.0;
  if (fl.on) {
    const float inv_n1 = 1.0f / (float)a.N1;
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int m = reps[i] >= 0 ? reps[i] : 0, r = mode_row(m, a.N1, inv_n1);
      wr[i] = wp[i] = flow_weight(fl, m - r * a.N1 - (a.N1 >> 1), r - (a.N2 >> 1));
    }
  } else if (a.mode_weight) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int rep = reps[i] >= 0 ? reps[i] : 0;
      wr[i] = a.mode_weight[rep];
      wp[i] = a.mode_weight[partners[i] >= 0 ? partners[i] : rep];
    }
  }
#pragma unroll
  for (int i = 0; i < N; ++i)
    e[i] = reps[i] >= 0 ? pair_energy_v<C>(fr[i], fp[i], wr[i], wp[i], partners[i] >= 0) : 0.0;
}

// Workgroup-wide sum / integer min / exclusive scan for NW
// waves (NW = 1: the wave operations alone, no barrier).  Every thread gets
// the result; the summation order is fixed.
template <int NW>
__device__ __forceinline__ double block_sum(double v, double *red, int wave) {
  v = wave_sum(v);
  if constexpr (NW == 1) {
    return v;
  } else {
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[wave] = v;
    __syncthreads();
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < NW; ++w) s += red[w];
    return s;
  }
}
template <int NW>
__device__ __forceinline__ int block_min_i(int v, int *red, int wave) {
  v = wave_min_i(v);
  if constexpr (NW == 1) {
    return v;
  } else {
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[wave] = v;
    __syncthreads();
    int s = INT_MAX;
#pragma unroll
    for (int w = 0; w < NW; ++w) s = min(s, red[w]);
    return s;
  }
}
template <int NW, typename V>
__device__ __forceinline__ V block_exclusive_scan(V v, V *red, int wave, int lane) {
  V x = wave_exclusive_scan<V>(v, lane);
  if constexpr (NW == 1) {
    return x;
  } else {
    const V tot = __shfl(x + v, 63, 64);
    __syncthreads();
    if (lane == 0) red[wave] = tot;
    __syncthreads();
    V base = V(0);
#pragma unroll
    for (int w = 0; w < NW; ++w)
      if (w < wave) base += red[w];
    return base + x;
  }
}

// Waves per SIMD asked of the compiler: four for up to four waves per cell (the
// unit energies stay in registers beside the sort's); the wide forms (below) need
// one workgroup per CU.
template <int NW>
constexpr int ems_min_waves() {
  return NW <= 4 ? 4 : (NW + 3) / 4;
}

// Sorted values in LDS: position j at j + j / 16, so that threads reading 16 (or 4)
// consecutive positions each fall on different banks.
__host__ __device__ __forceinline__ constexpr int ems_sidx(int j) { return j + (j >> 4); }

// Buckets of the value sort, two 16-bit counters per word: about 3,072, or two per
// sorted position for the small forms.  They take the unused tail of the sorted
// array where it is long enough, else LDS of their own.
template <int R, int NW>
constexpr int ems_bucket_words() {
  constexpr int w = (1536 + 64 * NW - 1) / (64 * NW);
  return 64 * NW * (w < R ? w : R);
}
template <int R, int NW>
__host__ __device__ __forceinline__ int ems_bucket_at(int J) {   // first word of the buckets
  constexpr int top = 2 * ems_sidx(64 * R * NW);
  const int own = 2 * ems_sidx(J + 1) + 2;
  return own + ems_bucket_words<R, NW>() <= top ? own : top;
}
template <int R, int NW>
__host__ __device__ __forceinline__ size_t ems_lds_bytes(int J) {
  const int top = 2 * ems_sidx(64 * R * NW), end = ems_bucket_at<R, NW>(J) + ems_bucket_words<R, NW>();
  return 4 * (size_t)(end > top ? end : top);
}

// A bucket with more values than this goes to the comparison network instead.
constexpr int EMS_BUCKET_MAX = 64;

// One workgroup of NW waves per cell.  Thread t holds the energies of units
// t, t + NT, ... in registers from the first load to the keep flags, so the
// coefficients are read once (a second read of the kept few gives the retained
// power).  The order of eq. (sorted_energy) is by energy, ties by ascending unit
// id.  Every quantity before the cut depends only on the sorted energy values, so
// the sort carries values only; which of several units tied at the cut energy are
// kept is settled afterwards by ascending id (a prefix count of the ties).
//
// The sort: non-negative FP64 values order as their bits, so the top 32 bits, scaled
// over the range present, give a bucket; one LDS counter per bucket, its scan, and a
// rank inside the bucket (a handful of values) place every value.  Zeros (modes
// outside a flow's propagating band) are the tail and take no bucket.  A crowded
// bucket (more than EMS_BUCKET_MAX values, for instance a flat spectrum's ties) or a
// negative weighted energy sends the cell to the comparison network instead: each wave sorts its 64 R values
// in registers and the runs are merged pairwise through LDS (merge path).
//
// What bounds it: latency and LDS work per cell (20,480 cells of 2,111 units: 0.76 GB of
// coefficients and masks).  With the network for every cell, each thread's units
// consecutive (64 cache lines per load) and the coefficients and a unit record per
// mode read again for the keep flags the launch took 0.88 ms; now 0.56 ms (and
// eight flow steps of 2,560 cells 1.31 to 0.53 ms).  A cell that falls back pays for both:
// equal amplitudes in every mode, 20,480 cells, 0.87 ms (0.89 with the network alone) at 2,111 units,
// 0.31 (0.235) at 512; four cells 27.2 us (24.6).
template <typename T, int R, int NW>
__global__ __launch_bounds__(64 * NW, (ems_min_waves<NW>())) void ems_kernel(EmsArgs a) {
  constexpr int NT = 64 * NW, JW = 64 * R, JP = JW * NW;
  extern __shared__ __align__(16) double sorted[];   // position j at ems_sidx(j)
  __shared__ double red0[NW], red1[NW];
  __shared__ int redi0[NW], redi1[NW];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, t = threadIdx.x;
  // cell: the output index; in flow mode step s of cell c is v = s n_cells_f + c
  // and reads the coefficients of cell c
  const int64_t cell = a.cell_begin + blockIdx.x;
  const int64_t fcell = a.flow ? cell % a.n_cells_f : cell;
  using C = typename vec2<T>::type;
  const C *f = reinterpret_cast<const C *>(a.f) + fcell * a.M;
  FlowRec fl{};
  fl.on = a.flow != nullptr;
  if (fl.on) {
    const double *fr = a.flow + 6 * cell;
    fl.ux = fr[0]; fl.uy = fr[1]; fl.N = fr[2]; fl.fc = fr[3]; fl.rho = fr[4]; fl.ks = fr[5];
  }
  const int J = a.J;

  // eq. (energy) / (weighted_e): e[r] is unit r NT + t (0 beyond J).  Batches of EB
  // units: few memory latencies per thread, few live registers.
  double e[R];
  double t1 = 0.0, t2 = 0.0;
  constexpr int EB = R < 4 ? R : 4;
  static_assert(R % EB == 0, "energy batches must divide R");
#pragma unroll
  for (int r0 = 0; r0 < R; r0 += EB) {
    int reps[EB], partners[EB];
#pragma unroll
    for (int i = 0; i < EB; ++i) {
      const int u = (r0 + i) * NT + t;
      const int2 un = a.units[u < J ? u : max(J - 1, 0)];
      reps[i] = u < J ? un.x : -1;
      partners[i] = un.y;
    }
    double eb[EB];
    batch_energy<C, EB>(a, fl, f, reps, partners, eb);
#pragma unroll
    for (int i = 0; i < EB; ++i) e[r0 + i] = eb[i];
  }
  // sums, and the range of the top words of the non-zero energies (a negative or
  // unordered one makes the minimum -1)
  int kmin = INT_MAX, nkmax = 0;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    t1 += e[r];
    t2 += e[r] * e[r];
    const int hi = __double2hiint(e[r]);
    if (e[r] != 0.0) {
      kmin = min(kmin, e[r] > 0.0 ? hi : -1);
      nkmax = min(nkmax, -hi);
    }
  }
  constexpr int BW = ems_bucket_words<R, NW>(), NB = 2 * BW, WPT = BW / NT;
  unsigned *bkt = reinterpret_cast<unsigned *>(sorted) + ems_bucket_at<R, NW>(J);
#pragma unroll
  for (int i = 0; i < WPT; ++i) bkt[i * NT + t] = 0u;
  double T1 = wave_sum(t1), T2 = wave_sum(t2);
  kmin = wave_min_i(kmin);
  nkmax = wave_min_i(nkmax);
  if (lane == 0) {
    red0[wave] = T1; red1[wave] = T2; redi0[wave] = kmin; redi1[wave] = nkmax;
  }
  __syncthreads();
  if constexpr (NW > 1) {
    T1 = T2 = 0.0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      T1 += red0[w];
      T2 += red1[w];
      kmin = min(kmin, redi0[w]);
      nkmax = min(nkmax, redi1[w]);
    }
  }

  // eq. (sorted_energy).  The bucket falls with the energy; a float product of the
  // (exactly converted or rounded, either way monotone) distance from the largest
  // keeps the order.
  int pos[R];   // bucket | place in the bucket << 16, or -1
  int crowd = 0;
  if (kmin >= 0) {
    const float scale = (float)NB / ((float)(-nkmax - kmin) + 1.0f) * 0.999999f;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      pos[r] = -1;
      if (e[r] != 0.0) {
        const int b = min(NB - 1, (int)((float)(-nkmax - __double2hiint(e[r])) * scale));
        const int sh = (b & 1) * 16;
        pos[r] = b | (int)((atomicAdd(&bkt[b >> 1], 1u << sh) >> sh) & 0xffffu) << 16;
      }
    }
    __syncthreads();
    unsigned wv[WPT];
    int sum = 0;
#pragma unroll
    for (int i = 0; i < WPT; ++i) {
      wv[i] = bkt[t * WPT + i];
      const int lo = wv[i] & 0xffff, hi = wv[i] >> 16;
      sum += lo + hi;
      crowd = max(crowd, max(lo, hi));
    }
    int run = block_exclusive_scan<NW, int>(sum, redi0, wave, lane);
#pragma unroll
    for (int i = 0; i < WPT; ++i) {   // counts become starts
      const int lo = wv[i] & 0xffff, hi = wv[i] >> 16;
      bkt[t * WPT + i] = (unsigned)run | (unsigned)(run + lo) << 16;
      run += lo + hi;
    }
    crowd = -block_min_i<NW>(-crowd, redi1, wave);
    if (t == NT - 1) redi0[0] = run;   // non-zero values
    __syncthreads();
  }
  if (kmin >= 0 && crowd <= EMS_BUCKET_MAX) {
    const int nnz = redi0[0];
    auto start = [&](int b) -> int { return b < NB ? (int)((bkt[b >> 1] >> ((b & 1) * 16)) & 0xffffu) : nnz; };
    // values in bucket order first, without the padding (position j at j)
#pragma unroll
    for (int r = 0; r < R; ++r)
      if (pos[r] >= 0) sorted[start(pos[r] & 0xffff) + (pos[r] >> 16)] = e[r];
    __syncthreads();
    // rank inside the bucket: values above, and equal ones at earlier places (a value
    // there need only exceed the next FP64 below e)
#pragma unroll
    for (int r = 0; r < R; ++r) {
      if (pos[r] < 0) continue;
      const int b = pos[r] & 0xffff, s0 = start(b), s1 = start(b + 1), mine = s0 + (pos[r] >> 16);
      int rank = s0;
      if (s1 - s0 > 1) {
        const double below = __longlong_as_double(__double_as_longlong(e[r]) - 1);
        for (int q = s0; q < s1; q += 2) {
          const double v0 = sorted[q], v1 = sorted[q + 1];   // (q + 1 <= J: inside the array)
          rank += v0 > (q < mine ? below : e[r]);
          rank += q + 1 < s1 && v1 > (q + 1 < mine ? below : e[r]);
        }
      }
      pos[r] = rank;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < R; ++r)
      if (pos[r] >= 0) sorted[ems_sidx(pos[r])] = e[r];
    for (int j = nnz + t; j < J; j += NT) sorted[ems_sidx(j)] = 0.0;
    __syncthreads();
  } else {
    // the comparison network: runs of JW per wave, then merges
    __syncthreads();
    double v[R];
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = e[r];
    wave_sort_desc<R>(v, lane);
#pragma unroll
    for (int r = 0; r < R; ++r) sorted[ems_sidx(t * R + r)] = v[r];
#pragma unroll 1
    for (int width = JW; width < JP; width *= 2) {
      __syncthreads();
      const int o0 = t * R;                       // first output position
      const int base = o0 / (2 * width) * (2 * width);
      // runs A = [base, base + width) and B = the rest of the pair (shorter, or
      // empty, at the end when NW is not a power of two)
      const int lb = min(width, max(0, JP - base - width));
      const int d = o0 - base;                    // outputs before mine in this merged run
      auto A = [&](int i) { return sorted[ems_sidx(base + i)]; };
      auto B = [&](int i) { return sorted[ems_sidx(base + width + i)]; };
      if (lb > 0) {
        int lo = d > lb ? d - lb : 0, hi = d < width ? d : width;
        while (lo < hi) {                         // first d outputs take lo from A
          const int mid = (lo + hi) >> 1;
          if (A(mid) >= B(d - 1 - mid)) lo = mid + 1;
          else hi = mid;
        }
        int ia = lo, ib = d - lo;
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const double va = A(min(ia, width - 1)), vb = B(min(ib, lb - 1));   // in bounds; guarded below
          const bool take_a = ib >= lb || (ia < width && va >= vb);
          v[r] = take_a ? va : vb;
          ia += take_a;
          ib += !take_a;
        }
      } else {                                    // unpaired run: already in place
#pragma unroll
        for (int r = 0; r < R; ++r) v[r] = sorted[ems_sidx(o0 + r)];
      }
      __syncthreads();
#pragma unroll
      for (int r = 0; r < R; ++r) sorted[ems_sidx(o0 + r)] = v[r];
    }
    __syncthreads();
  }

  const int Jmax = J < a.k_max ? J : a.k_max;
  // eq. (n_eff) over all J units, clipped by the budget
  const double neff = T2 > 0.0 ? T1 * T1 / T2 : 0.0;
  const double nclip = neff < (double)Jmax ? neff : (double)Jmax;
  // eq. (s_delta) over the first J_max - 1 gaps
  double sd = 0.0;
  for (int j = t; j < Jmax - 1; j += NT) {
    const double ea = sorted[ems_sidx(j)], eb = sorted[ems_sidx(j + 1)];
    double term;
    if (eb == 0.0 && ea == 0.0) term = 1.0;
    else if (eb == 0.0) term = 0.0;
    else term = exp(-(ea / eb - 1.0) / a.delta);
    sd += term;
  }
  // eq. (f_cum): running sum in sorted order, thread t at positions t R .. t R + R - 1
  double loc = 0.0;
#pragma unroll
  for (int r = 0; r < R; ++r)
    if (t * R + r < J) loc += sorted[ems_sidx(t * R + r)];
  const double sdsum = block_sum<NW>(sd, red0, wave);
  const double sdel = Jmax < 2 ? 1.0 : sdsum / (double)(Jmax - 1);
  // eqs. (c_score), (alpha_c)
  const double Cs = (Jmax > 0 ? a.w1 * nclip / (double)Jmax : 0.0) + a.w2 * sdel;
  const double alphaC = a.alpha_min + (a.alpha_max - a.alpha_min) * Cs;
  // the first K with theta(K) >= alpha_C
  const double run0 = block_exclusive_scan<NW, double>(loc, red1, wave, lane);
  int kc = INT_MAX;
  // (a division only near the crossing: below `under` the quotient is short of alpha_C;
  // non-negative energies cross a positive alpha_C once, in the one thread whose sums
  // straddle it.  alpha_C <= 0, where alpha_min > alpha_max and C > 1, is met by the first
  // position and straddled by no thread's sums: there, and with negative weighted
  // energies, every position is divided)
  const bool every = kmin < 0 || !(alphaC > 0.0);
  const double under = alphaC * T1 * (1.0 - 1e-12), over = alphaC * T1 * (1.0 + 1e-12);
  if (T1 > 0.0 && t * R < J && (every || (run0 + loc >= under && run0 <= over))) {
    double v[R], run = run0;
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = sorted[ems_sidx(t * R + r)];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      run += v[r];
      if (kc == INT_MAX && t * R + r < J && (every || !(run < under)) && run / T1 >= alphaC) kc = t * R + r + 1;
    }
  }
  kc = block_min_i<NW>(kc, redi0, wave);
  // eq. (k_elastic)
  int kstar;
  if (!(T1 > 0.0)) {
    kstar = a.k_min < J ? a.k_min : J;
  } else {
    const int kcc = kc == INT_MAX ? J : kc;
    const int k = kcc > a.k_min ? kcc : a.k_min;
    kstar = k < Jmax ? k : Jmax;
  }
  // cut energy E_(K*), the retained sum of the first K* sorted energies, and
  // how many units lie strictly above the cut or at it
  const double eth = kstar > 0 ? sorted[ems_sidx(kstar - 1)] : 0.0;
  double part = 0.0;
  int cgt = 0;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int j = t * R + r, u = r * NT + t;
    if (j < kstar) part += sorted[ems_sidx(j)];
    if (u < J) cgt += (e[r] > eth) + ((e[r] == eth) << 16);   // at most 4,096 of each
  }
  double th = wave_sum(part);
  int cnt = wave_sum_i(cgt);
  if constexpr (NW > 1) {
    __syncthreads();
    if (lane == 0) { red0[wave] = th; redi1[wave] = cnt; }
    __syncthreads();
    th = 0.0;
    cnt = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) { th += red0[w]; cnt += redi1[w]; }
  }
  const int need = kstar - (cnt & 0xffff);   // units kept at the cut energy, lowest ids first
  const int neq = cnt >> 16;

  // Ties straddling the cut (more units at the cut energy than kept there):
  // rank the tied units by id.  Otherwise every unit at the cut is kept.
  unsigned kept = 0;   // bit r: unit r NT + t is kept
  if (kstar > 0 && neq > need) {   // the same in every thread
    int before = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const bool tie = r * NT + t < J && e[r] == eth;
      const uint64_t m = __ballot(tie);
      int rank = before + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
      int total = __popcll(m);
      if constexpr (NW > 1) {
        __syncthreads();
        if (lane == 0) redi0[wave] = total;
        __syncthreads();
        total = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
          if (w < wave) rank += redi0[w];
          total += redi0[w];
        }
      }
      before += total;
      if (r * NT + t < J && (e[r] > eth || (tie && rank < need))) kept |= 1u << r;
    }
  } else if (kstar > 0) {
#pragma unroll
    for (int r = 0; r < R; ++r)
      if (r * NT + t < J && e[r] >= eth) kept |= 1u << r;
  }

  // keep flags and the retained power: consecutive lanes take consecutive units, whose
  // representatives ascend and partners descend by one, so the byte stores coalesce
  double pw = 0.0;
  uint8_t *kout = a.keep ? a.keep + cell * a.M : nullptr;   // flow mode may skip the masks
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int u = r * NT + t;
    if (u >= J) continue;
    const bool k = (kept >> r) & 1u;
    if (!kout && !k) continue;
    const int2 un = a.units[u];
    if (kout) {
      kout[un.x] = k;
      if (un.y >= 0) kout[un.y] = k;
    }
    if (k) {
      const C fa = f[un.x];
      pw += (double)fa.x * (double)fa.x + (double)fa.y * (double)fa.y;
      if (un.y >= 0) {
        const C fb = f[un.y];
        pw += (double)fb.x * (double)fb.x + (double)fb.y * (double)fb.y;
      }
    }
  }
  if (kout && t == 0 && a.dc >= 0) kout[a.dc] = 0;   // the excluded mode belongs to no unit
  const double P = block_sum<NW>(pw, red1, wave);
  if (t == 0) {
    a.k_star[cell] = kstar;
    double *st = a.stats + cell * 8;
    st[0] = T1; st[1] = P; st[2] = neff; st[3] = sdel;
    st[4] = Cs; st[5] = alphaC; st[6] = T1 > 0.0 ? th / T1 : 0.0; st[7] = (double)J;
  }
}

// Units on the host: +-k pairs (representative k_y > 0, or k_y = 0 and k_x > 0)
// when both members lie in the box, otherwise single modes; ascending id.
static void build_units(int N1, int N2, bool pairs, bool exclude_dc, std::vector<int2> &out) {
  out.clear();
  const int lo1 = -(N1 / 2), lo2 = -(N2 / 2), hi1 = lo1 + N1 - 1, hi2 = lo2 + N2 - 1;
  for (int r = 0; r < N2; ++r) {
    for (int i = 0; i < N1; ++i) {
      const int kx = lo1 + i, ky = lo2 + r, idx = r * N1 + i;
      const bool dc = kx == 0 && ky == 0;
      if (dc && exclude_dc) continue;
      int partner = -1;
      if (pairs && !dc) {
        const int mx = -kx, my = -ky;
        if (mx >= lo1 && mx <= hi1 && my >= lo2 && my <= hi2) partner = (my - lo2) * N1 + (mx - lo1);
      }
      if (partner >= 0 && !(ky > 0 || (ky == 0 && kx > 0))) continue;
      out.push_back(make_int2(idx, partner));
    }
  }
}


enufft_status ems_units(enufft_plan_t p, const enufft_ems_params *prm, UnitTable **ut) {
  UnitTable &u = p->units[prm->use_pairs ? 1 : 0][prm->exclude_dc ? 1 : 0];
  if (!u.built) {
    std::vector<int2> v;
    build_units(p->N1, p->N2, prm->use_pairs != 0, prm->exclude_dc != 0, v);
    const int M = p->N1 * p->N2;
    u.J = (int)v.size();
    // the kernel's branch-free loads read unit max(J - 1, 0): give an empty set
    // one harmless entry (mode 0, no partner) that is never counted
    if (v.empty()) v.push_back(make_int2(0, -1));
    std::vector<int4> of_mode(M, make_int4(-1, -1, -1, 0));
    for (int i = 0; i < u.J; ++i) {
      of_mode[v[i].x] = make_int4(v[i].x, v[i].y, i, 0);
      if (v[i].y >= 0) of_mode[v[i].y] = make_int4(v[i].x, v[i].y, i, 0);
    }
    u.Jpad = 64;
    while (u.Jpad < u.J) u.Jpad <<= 1;
    void *d = nullptr, *dm = nullptr;
    hipError_t e = hipMalloc(&d, std::max<size_t>(1, v.size()) * sizeof(int2));
    if (e == hipSuccess) p->allocations.push_back(d);
    if (e == hipSuccess) e = hipMalloc(&dm, (size_t)M * sizeof(int4));
    if (e == hipSuccess) p->allocations.push_back(dm);
    if (e != hipSuccess) {
      p->last_error = "EMS unit table allocation failed";
      return ENUFFT_ENOMEM;
    }
    if (!v.empty()) e = hipMemcpy(d, v.data(), v.size() * sizeof(int2), hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemcpy(dm, of_mode.data(), (size_t)M * sizeof(int4), hipMemcpyHostToDevice);
    if (e != hipSuccess) {
      p->last_error = std::string("EMS unit table upload: ") + hipGetErrorString(e);
      p->faulted = true;
      return ENUFFT_EDEVICE;
    }
    u.d_units = (int2 *)d;
    u.d_mode_unit = (int4 *)dm;
    u.built = true;
  }
  *ut = &u;
  return ENUFFT_OK;
}

enufft_status ems_validate(enufft_plan_t p, const void *f, const enufft_ems_params *prm, uint8_t *keep,
                           int32_t *k_star, double *stats) {
  auto bad = [&](const char *m) {
    p->last_error = std::string("enufft_ems: ") + m;
    return ENUFFT_EINVAL;
  };
  if (!prm) return bad("null params");
  if (!f || !keep || !k_star || !stats) return bad("null output or input pointer");
  if (prm->k_min < 0 || prm->k_max < 1 || prm->k_min > prm->k_max) return bad("need 0 <= k_min <= k_max, k_max >= 1");
  if (!(prm->alpha_min >= 0.0 && prm->alpha_min <= 1.0 && prm->alpha_max >= 0.0 && prm->alpha_max <= 1.0))
    return bad("alpha_min and alpha_max must be in [0, 1]");
  if (!(prm->delta > 0.0) || !std::isfinite(prm->delta)) return bad("delta must be > 0");
  if (!(prm->w1 >= 0.0 && prm->w1 <= 1.0 && prm->w2 >= 0.0 && prm->w2 <= 1.0)) return bad("w1, w2 must be in [0, 1]");
  if ((prm->use_pairs != 0 && prm->use_pairs != 1) || (prm->exclude_dc != 0 && prm->exclude_dc != 1))
    return bad("use_pairs and exclude_dc must be 0 or 1");
  return ENUFFT_OK;
}

// Whether a launch of `blocks` cells leaves the CUs mostly idle with the narrow
// forms (fewer than eight of their waves per CU): then the wide forms.
// ENUFFT_EMS_WIDE=0 or 1 forces the choice.
bool ems_wide(const enufft_plan_t p, int J, int64_t blocks) {
  if (const char *ev = std::getenv("ENUFFT_EMS_WIDE")) return std::atoi(ev) != 0;
  const int64_t waves = blocks * ((J + 1023) / 1024);
  return waves < (int64_t)p->n_cu * 8;
}

template <typename T, int R, int NW>
static hipError_t launch_ems_form(const EmsArgs &a, int J, int blocks, hipStream_t s) {
  hipLaunchKernelGGL((ems_kernel<T, R, NW>), dim3(blocks), dim3(64 * NW), (ems_lds_bytes<R, NW>(J)), s, a);
  return hipGetLastError();
}

// The form of a cell: the smallest 64 R NW >= J, R values a lane (a power of two up to
// 16) and NW waves (up to 4), or the wide forms' four values and up to 16 waves.
template <typename T>
hipError_t launch_ems_t(const EmsArgs &a, int J, int blocks, hipStream_t s, bool wide) {
  if (wide && J > 256) {
    // few cells: each cell's latency is the launch's, so more waves per cell, four
    // values per lane
    if (J <= 512) return launch_ems_form<T, 4, 2>(a, J, blocks, s);
    if (J <= 768) return launch_ems_form<T, 4, 3>(a, J, blocks, s);
    if (J <= 1024) return launch_ems_form<T, 4, 4>(a, J, blocks, s);
    if (J <= 1536) return launch_ems_form<T, 4, 6>(a, J, blocks, s);
    if (J <= 2048) return launch_ems_form<T, 4, 8>(a, J, blocks, s);
    if (J <= 3072) return launch_ems_form<T, 4, 12>(a, J, blocks, s);
    if (J <= 4096) return launch_ems_form<T, 4, 16>(a, J, blocks, s);
    return hipErrorInvalidValue;
  }
  if (J <= 64) return launch_ems_form<T, 1, 1>(a, J, blocks, s);
  if (J <= 128) return launch_ems_form<T, 2, 1>(a, J, blocks, s);
  if (J <= 256) return launch_ems_form<T, 4, 1>(a, J, blocks, s);
  if (J <= 512) return launch_ems_form<T, 8, 1>(a, J, blocks, s);
  if (J <= 1024) return launch_ems_form<T, 16, 1>(a, J, blocks, s);
  if (J <= 2048) return launch_ems_form<T, 16, 2>(a, J, blocks, s);
  if (J <= 3072) return launch_ems_form<T, 16, 3>(a, J, blocks, s);
  if (J <= 4096) return launch_ems_form<T, 16, 4>(a, J, blocks, s);
  return hipErrorInvalidValue;
}

enufft_status record_start(enufft_plan_t p, int kind, hipEvent_t *ev);
enufft_status record_stop(enufft_plan_t p, int kind, hipEvent_t start);

enufft_status ems_launch(enufft_plan_t p, const void *f, const enufft_ems_params *prm, const double *mode_weight,
                         uint8_t *keep, int32_t *k_star, double *stats, int64_t cell_begin, int64_t cell_count) {
  UnitTable *ut = nullptr;
  enufft_status st = ems_units(p, prm, &ut);
  if (st != ENUFFT_OK) return st;
  if (ut->Jpad > 4096)   // beyond the per-cell register sort: device sort per cell
    return big_ems(p, f, prm, mode_weight, keep, k_star, stats, ut, cell_begin, cell_count);
  EmsArgs a{};
  a.f = f; a.mode_weight = mode_weight; a.keep = keep; a.k_star = k_star; a.stats = stats;
  a.units = ut->d_units; a.J = ut->J;
  a.dc = prm->exclude_dc ? (p->N2 / 2) * p->N1 + p->N1 / 2 : -1;
  a.M = p->N1 * p->N2;
  a.N1 = p->N1; a.N2 = p->N2;
  a.cell_begin = cell_begin;
  a.cell_end = cell_begin + cell_count;
  a.k_min = prm->k_min; a.k_max = prm->k_max;
  a.alpha_min = prm->alpha_min; a.alpha_max = prm->alpha_max; a.delta = prm->delta;
  a.w1 = prm->w1; a.w2 = prm->w2;
  const int blocks = (int)cell_count;
  const bool wide = ems_wide(p, ut->J, blocks);
  hipError_t e = p->prec == ENUFFT_F64 ? launch_ems_t<double>(a, ut->J, blocks, p->stream, wide)
                                       : launch_ems_t<float>(a, ut->J, blocks, p->stream, wide);
  if (e != hipSuccess) {
    p->last_error = std::string("EMS launch: ") + hipGetErrorString(e);
    p->faulted = true;
    return ENUFFT_EDEVICE;
  }
  return ENUFFT_OK;
}

}  // namespace enufft

extern "C" enufft_status enufft_ems(enufft_plan_t p, const void *f, const enufft_ems_params *prm,
                                    const double *mode_weight, uint8_t *keep, int32_t *k_star, double *stats) {
  if (!p) return ENUFFT_EINVAL;
  if (p->faulted) {
    p->last_error = "enufft_ems: plan unusable after a device fault";
    return ENUFFT_ESTATE;
  }
  enufft_status st = enufft::ems_validate(p, f, prm, keep, k_star, stats);
  if (st != ENUFFT_OK) return st;
  if (p->n_cells == 0) return ENUFFT_OK;
  hipEvent_t ev;
  st = enufft::record_start(p, 1, &ev);
  if (st != ENUFFT_OK) return st;
  st = enufft::ems_launch(p, f, prm, mode_weight, keep, k_star, stats, 0, p->n_cells);
  if (st != ENUFFT_OK) return st;
  return enufft::record_stop(p, 1, ev);
}

extern "C" enufft_status enufft_ems_flow(enufft_plan_t p, const void *f, const enufft_ems_params *prm,
                                         int32_t n_steps, const double *flow, uint8_t *keep, int32_t *k_star,
                                         double *stats) {
  if (!p) return ENUFFT_EINVAL;
  if (p->faulted) {
    p->last_error = "enufft_ems_flow: plan unusable after a device fault";
    return ENUFFT_ESTATE;
  }
  uint8_t dummy = 0;
  // the masks are optional here: validate with a stand-in pointer
  enufft_status st = enufft::ems_validate(p, f, prm, keep ? keep : &dummy, k_star, stats);
  if (st != ENUFFT_OK) return st;
  if (n_steps < 1 || !flow) {
    p->last_error = "enufft_ems_flow: need n_steps >= 1 and flow records";
    return ENUFFT_EINVAL;
  }
  if (p->n_cells == 0) return ENUFFT_OK;
  if ((int64_t)n_steps * p->n_cells > (int64_t)INT32_MAX) {
    p->last_error = "enufft_ems_flow: n_steps * n_cells above 2^31 - 1";
    return ENUFFT_EINVAL;
  }
  enufft::UnitTable *ut = nullptr;
  st = enufft::ems_units(p, prm, &ut);
  if (st != ENUFFT_OK) return st;
  if (ut->Jpad > 4096) {
    p->last_error = "enufft_ems_flow: more than 4096 units per cell is not supported";
    return ENUFFT_EUNSUPPORTED;
  }
  enufft::EmsArgs a{};
  a.f = f; a.mode_weight = nullptr; a.flow = flow; a.n_cells_f = p->n_cells;
  a.keep = keep; a.k_star = k_star; a.stats = stats;
  a.units = ut->d_units; a.J = ut->J;
  a.dc = prm->exclude_dc ? (p->N2 / 2) * p->N1 + p->N1 / 2 : -1;
  a.M = p->N1 * p->N2;
  a.N1 = p->N1; a.N2 = p->N2;
  a.cell_begin = 0;
  a.cell_end = (int64_t)n_steps * p->n_cells;
  a.k_min = prm->k_min; a.k_max = prm->k_max;
  a.alpha_min = prm->alpha_min; a.alpha_max = prm->alpha_max; a.delta = prm->delta;
  a.w1 = prm->w1; a.w2 = prm->w2;
  hipEvent_t ev;
  st = enufft::record_start(p, 1, &ev);
  if (st != ENUFFT_OK) return st;
  const int blocks = (int)a.cell_end;
  const bool wide = enufft::ems_wide(p, ut->J, blocks);
  hipError_t e = p->prec == ENUFFT_F64 ? enufft::launch_ems_t<double>(a, ut->J, blocks, p->stream, wide)
                                       : enufft::launch_ems_t<float>(a, ut->J, blocks, p->stream, wide);
  if (e != hipSuccess) {
    p->last_error = std::string("enufft_ems_flow launch: ") + hipGetErrorString(e);
    p->faulted = true;
    return ENUFFT_EDEVICE;
  }
  return enufft::record_stop(p, 1, ev);
}
