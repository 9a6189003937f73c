// Band-limited rows: the sum over the grid's bins as a sum over fewer, wider-spaced frequencies.
//
// A point's model E(f) = exp(-2 pi i (sum_m a_m g_m(f) + f T)) is a chirp: around f it is a tone of
// "time" t(f) = sum_m a_m g_m'(f) + T, and over a range of frequencies where |t(f) - t0| <= tb it
// is determined by its values on a uniform grid of step h = 1 / (2 sigma tb), sigma > 1 (the
// sampling theorem with oversampling sigma):
//   E(f_k) = sum_q K((f_k - f_q) / h) exp(-2 pi i t0 (f_k - f_q)) E(f_q),
// K a sinc windowed by the "exponential of semicircle" exp(beta (sqrt(1 - (2x/w)^2) - 1)) of
// Barnett, Magland and af Klinteberg (SIAM J. Sci. Comput. 41, 2019), w nodes wide. With w from
// Kaiser's estimate for 300 dB and beta = 0.98 pi (w/2) (1 - 1/sigma) the largest error over the
// band is about 1e-14 (root mean square 3e-15): below the rounding of a phase of hundreds of
// cycles. So the data side can be summed once per event, U_q = sum_k u_k K(..) exp(..), and
// Z_det = sum_k u_k E_det(f_k) = sum_q U_q E_det(f_q) for every point whose t(f) stays inside
// [t0 - tb, t0 + tb] on the rows' frequencies, with the same error in the adjoint's moments (f E
// and g_m E are as band-limited as E).
//
// The grid is cut into panels (geometric in f) and a few wide segments from a panel to the top;
// each has candidate row sets (bands) for a range of (t0, tb). The set-up of a group of 64 points
// bounds t(f) over the group and takes, per segment, the band with the fewest rows that holds
// it, or the grid's own bins where none does: a group's plan.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "gwl_common.h"

namespace gwl {

constexpr int MAXPANEL = 14;    // panels of the grid
constexpr int MAXSEG = 20;      // panels and wide segments
constexpr int MAXBRK = 63;      // frequency intervals on which t(f) is bounded
constexpr int MAXCAND = 512;    // bands of all segments
constexpr int PLAN_INTS = 64;   // a group's plan: rows in all, pieces, float64 path, rows per chunk;
                                // then per piece its first row, its rows and its band (-1: bins)
constexpr int MAXLEV = 3;       // levels: fixed choices of bands, from which a point alone takes its rows
constexpr double BAND_FILL = 0.98;  // share of a band's half-width that a group may use
// A calibrated event's rows lie at most a quarter of the frequency, and CAL_REACH node spacings (in ln f, hx
// each), beyond their interval: cal_reach spacings. The interval's Catmull-Rom cubic, run on x spacings beyond,
// has slope weights (1 + 4x + 3x^2) / 2, (1 - 6x - 6x^2) / 2 and (2x + 3x^2) / 2 on the differences of the
// nodes around it, whose magnitudes add to 6x (1 + x) from x = 0.2 on and to 1.5 at most up to there and within the
// interval: cal_slope times the largest difference bounds the slope per spacing.
constexpr double CAL_REACH = 0.75;
inline double cal_reach(double hx) { return fmin(0.22314355131420976 / hx, CAL_REACH); }   // ln 1.25
inline double cal_slope(double reach) { return fmax(1.5, 6.0 * reach * (1.0 + reach)); }

// Rows that a group of a call may have and still walk them in float64: any number in a float64 call; in a
// mixed-precision one as many as take the time of its M bins in mixed precision. Measured on every bin, float64 to mixed (three
// detectors, 8 s; 65,536 values, 16,384 gradients, and with 10 calibration nodes 16,384 and 8,192): 1,553 and 1,403 us,
// 696 and 545, 991 and 708, 824 and 659.
__host__ __device__ inline int float64_most(bool mixed, bool grad, bool cal, int64_t M) {
  return mixed ? (int)(M * (cal ? (grad ? 80 : 71) : (grad ? 78 : 90)) / 100) : 0x7fffffff;
}

struct BandCand {
  double t0, tb;      // centre and half-width of the band (s)
  double step;        // spacing of its rows (Hz)
  int row0, rows;     // its rows in the event's tables
  int i0, i1;         // the intervals that its rows' frequencies reach over
};
// A level: a fixed choice of bands (and bins), in the form of a group's plan, and the interval limits within
// which t(f) has to lie for them to hold a point. Live-length calls walk levels: which of the batch's points are
// live, and what the rows past them hold, must not show in a point's bits.
struct BandLevel {
  int rows, np;
  int row0[MAXPANEL + 2], n[MAXPANEL + 2];   // per piece its first row, its rows
  double step[MAXPANEL + 2];                 // and their spacing (Hz)
  double2 lim[MAXBRK + 1];                   // lowest and highest t per interval
};
struct BandHead {
  int nbrk, ncand, nseg, npanel;
  int nlev[2];             // levels of a float64 and of a mixed-precision call (fewest rows first)
  int c0[MAXSEG + 1];      // each segment's bands, fewest rows first
  int first[MAXSEG];       // the panel that a segment starts with
  int k0[MAXSEG];          // its bins
  int bins[MAXSEG];
  alignas(16) double gp[MAXBRK + 1][NBASIS];  // g_m'(f) at the interval ends (each g_m' is monotone between them)
  BandCand cand[MAXCAND];
  BandLevel lev[MAXLEV + 1];   // the last: every bin, for a point that no level holds
};

// How a band's rows are made (host to device, at event creation).
struct BandGen {
  int src0, nsrc;     // the rows that it sums: a segment's bins, or the segment's widest band's rows
  int src_half;       // their spacing in half bins (bins: 2; on a grid that is not uniform their
                      // frequencies are read instead)
  int half;           // its own spacing in half bins
  int n0;             // first row at fa + n0 h, fa the first source row's frequency
  int w;              // window width in rows
  int row0, rows;
  int klen;           // kernel values kept from koff, by half-bin distance (0: computed as needed)
  int64_t koff;
  double h, fa, t0, beta;
  double hdf;         // half a bin (Hz)
};

struct BandLds {
  float2 r[MAXBRK + 1];                      // lowest and highest t per interval over the group
  unsigned long long ok[MAXCAND / 64 + 1];   // bands that hold the group
  int plan[PLAN_INTS];
};
struct LevelLds {                            // in its place where points take levels
  double2 lim[MAXLEV][MAXBRK + 1];           // the levels' limits
  unsigned long long fit[MAXLEV];            // the points that each level holds
};

template <int CTRL>
__device__ inline float dpp_max(float v) {
  const int o = __builtin_amdgcn_update_dpp(__float_as_int(v), __float_as_int(v), CTRL, 0xf, 0xf, false);
  return fmaxf(v, __int_as_float(o));
}
// the largest of 64 lanes, in lane 63: within rows of 16, then across rows
__device__ inline float wave_max_hi(float v) {
  v = dpp_max<0x111>(v);  // row_shr:1
  v = dpp_max<0x112>(v);
  v = dpp_max<0x114>(v);
  v = dpp_max<0x118>(v);
  v = dpp_max<0x142>(v);  // row_bcast:15
  return dpp_max<0x143>(v);  // row_bcast:31
}

// sums over the lanes up to each of the first 16, and v one lane up (0 in lane 0)
template <int CTRL>
__device__ inline int dpp_or_zero(int v) {
  return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, false);
}
__device__ inline int sums_16(int v) {
  v += dpp_or_zero<0x111>(v);  // row_shr:1
  v += dpp_or_zero<0x112>(v);
  v += dpp_or_zero<0x114>(v);
  return v + dpp_or_zero<0x118>(v);
}
__device__ inline int lane_up(int v) { return dpp_or_zero<0x111>(v); }

// The steps are a chain of short reads by few wavefronts, bound by latency. They read what they need of the
// head without waiting for memory in turn: the slopes go to LDS while the point model runs, the bands
// and segments to registers before it, and a band's extremes come from two windows instead of a loop over
// its intervals. The multi-event set-up (330 groups of 12 events) went from 21.1 to 16.7 us with this,
// the calibrated one (256 groups, 20 node values a detector, copied by the two wavefronts that the
// point model leaves idle) from 20.4 to 17.5.

// Step 0, before a barrier, by the workgroup's threads from `first` on: the slopes. `slopes_s` holds
// BAND_LDS doubles, later the bands' first rows and rows.
constexpr int BAND_LDS = (MAXBRK + 1) * NBASIS;
static_assert(sizeof(int2) * MAXCAND <= sizeof(double) * BAND_LDS, "the bands' rows take the slopes' place");
__device__ inline void band_load(const BandHead* __restrict__ bh, double* slopes_s, int first = 0) {
  const double2* src = reinterpret_cast<const double2*>(&bh->gp[0][0]);
  double2* dst = reinterpret_cast<double2*>(slopes_s);
  for (int i = (int)threadIdx.x - first; i < BAND_LDS / 2; i += (int)blockDim.x - first) dst[i] = src[i];
}

// With levels, beside the slopes, by the same threads: their limits (read from memory on the way, they kept every
// wavefront waiting once an interval).
__device__ inline void level_load(const BandHead* __restrict__ bh, int nlev, LevelLds& s, int first) {
  for (int i = (int)threadIdx.x - first; i < nlev * (MAXBRK + 1); i += (int)blockDim.x - first)
    (&s.lim[0][0])[i] = bh->lev[i / (MAXBRK + 1)].lim[i % (MAXBRK + 1)];
}

// A lane's band (the first of its turns in step 2) and segment (step 3), requested ahead.
struct BandPre {
  BandCand cand;
  int ncand, nbrk, nseg, npanel, c0, nc, first, k0, bins;
};
__device__ __forceinline__ BandPre band_fetch(const BandHead* __restrict__ bh, int w, int lane) {
  BandPre f;
  const int c = w * WAVE + lane, j = lane < MAXSEG ? lane : MAXSEG - 1;
  f.cand = bh->cand[c < MAXCAND ? c : MAXCAND - 1];
  f.ncand = bh->ncand;
  f.nbrk = bh->nbrk;
  f.nseg = bh->nseg;
  f.npanel = bh->npanel;
  f.c0 = bh->c0[j];
  f.nc = bh->c0[j + 1] - f.c0;
  f.first = bh->first[j];
  f.k0 = bh->k0[j];
  f.bins = bh->bins[j];
  return f;
}

// Bounds of each point's t(f) over the intervals [w nbrk / nw, (w + 1) nbrk / nw): fn(interval, low, high).
// Every g_m' is monotone, so over an interval t lies within (t_i + t_i+1 -+ sum_m |a_m| |change of g_m'|) / 2.
// `slope`: a further phase, of at most `slope` cycles per unit of ln f.
template <int ND, class Fn>
__device__ __forceinline__ void band_bounds(const double* slopes_s, int nbrk, const double (&a)[NBASIS],
                                            const double (&T)[ND], int w, int nw, double slope, Fn fn) {
  double tlo = T[0], thi = T[0];
#pragma unroll
  for (int d = 1; d < ND; ++d) {
    tlo = fmin(tlo, T[d]);
    thi = fmax(thi, T[d]);
  }
  const int i0 = w * nbrk / nw, i1 = (w + 1) * nbrk / nw;
  double g[NBASIS], t = 0.0;
#pragma unroll
  for (int m = 0; m < NBASIS; ++m) {
    g[m] = slopes_s[i0 * NBASIS + m];
    t = fma(a[m], g[m], t);
  }
#pragma unroll 2
  for (int i = i0; i < i1; ++i) {
    double t1 = 0.0, v = 2.0 * slope * g[4];                   // g_4 = ln f
#pragma unroll
    for (int m = 0; m < NBASIS; ++m) {
      const double gn = slopes_s[(i + 1) * NBASIS + m];
      t1 = fma(a[m], gn, t1);
      v = fma(fabs(a[m]), fabs(gn - g[m]), v);
      g[m] = gn;
    }
    const double mid = t + t1;
    t = t1;
    fn(i, fma(0.5, mid - v, tlo), fma(0.5, mid + v, thi));
  }
}

// Step 1, by nw wavefronts that each hold the group's 64 points: bounds of t(f) over the group, each
// wavefront on its share of the intervals. Points with a NaN coefficient do not count (their value is NaN on
// any rows).
template <int ND>
__device__ inline void band_ranges(const double* slopes_s, int nbrk, const double (&a)[NBASIS], const double (&T)[ND],
                                   int w, int nw, int lane, BandLds& s, double slope = 0.0) {
  band_bounds<ND>(slopes_s, nbrk, a, T, w, nw, slope, [&](int i, double l, double h) {
    float hi = (float)h, nlo = -(float)l;
    const bool nan = !(hi == hi) || !(nlo == nlo);
    hi = wave_max_hi(nan ? -__builtin_inff() : hi);
    nlo = wave_max_hi(nan ? -__builtin_inff() : nlo);
    if (lane == WAVE - 1) s.r[i] = make_float2(-nlo, hi);
  });
}

// In its place for levels: the points that each level holds, by their own t(f) alone, into s.fit (all ones
// before). A NaN fits: its point's value is NaN on any rows.
template <int ND>
__device__ inline void band_fit(int nlev, int nbrk, const double* slopes_s, const double (&a)[NBASIS],
                                const double (&T)[ND], int w, int nw, int lane, LevelLds& s) {
  bool ok[MAXLEV];
#pragma unroll
  for (int l = 0; l < MAXLEV; ++l) ok[l] = true;
  band_bounds<ND>(slopes_s, nbrk, a, T, w, nw, 0.0, [&](int i, double lo, double hi) {
#pragma unroll
    for (int l = 0; l < MAXLEV; ++l) {
      if (l >= nlev) break;
      const double2 m = s.lim[l][i];
      ok[l] = ok[l] && !(lo < m.x) && !(hi > m.y);
    }
  });
#pragma unroll
  for (int l = 0; l < MAXLEV; ++l) {
    const unsigned long long m = __ballot(ok[l]);
    if (l < nlev && lane == 0) atomicAnd(&s.fit[l], m);
  }
}

// Step 2, after a barrier: the bands that hold the group, 64 per wavefront and turn. Lane i holds the
// extremes over 1, 2, 4, .. 32 intervals from i on; two such windows cover a band's intervals.
__device__ inline void band_hold(const BandHead* __restrict__ bh, const BandPre& own, double* slopes_s, int w, int nw,
                                 int lane, BandLds& s) {
  constexpr int NL = 6;
  static_assert(MAXBRK < (1 << NL), "window levels");
  float lo[NL], hi[NL];
  const float2 r = lane < own.nbrk ? s.r[lane] : make_float2(__builtin_inff(), -__builtin_inff());
  lo[0] = r.x;
  hi[0] = r.y;
#pragma unroll
  for (int l = 1; l < NL; ++l) {
    lo[l] = fminf(lo[l - 1], __shfl_down(lo[l - 1], 1 << (l - 1)));
    hi[l] = fmaxf(hi[l - 1], __shfl_down(hi[l - 1], 1 << (l - 1)));
  }
  int2* rows_s = reinterpret_cast<int2*>(slopes_s);
  for (int wd = w; wd * WAVE < own.ncand; wd += nw) {
    const int c = wd * WAVE + lane;
    const BandCand b = wd == w ? own.cand : bh->cand[c < MAXCAND ? c : MAXCAND - 1];
    const int len = b.i1 - b.i0 + 1, lv = len > 1 ? 31 - __clz(len) : 0, j = b.i1 + 1 - (1 << lv);
    float l0 = 0.0f, h0 = 0.0f;
#pragma unroll
    for (int l = 0; l < NL; ++l) {
      const float x = fminf(__shfl(lo[l], b.i0 & 63), __shfl(lo[l], j & 63));
      const float y = fmaxf(__shfl(hi[l], b.i0 & 63), __shfl(hi[l], j & 63));
      l0 = l == lv ? x : l0;
      h0 = l == lv ? y : h0;
    }
    const double lim = BAND_FILL * b.tb;
    const bool ok = c < own.ncand && (double)h0 - b.t0 <= lim && b.t0 - (double)l0 <= lim;
    if (c < MAXCAND) rows_s[c] = make_int2(b.row0, b.rows);
    const unsigned long long m = __ballot(ok);
    if (lane == 0) s.ok[wd] = m;
  }
}

// The band of segment `lane` that holds the group with the fewest rows (-1: none).
__device__ inline int band_of_segment(const BandPre& own, int lane, const BandLds& s) {
  if (lane >= own.nseg || own.nc == 0) return -1;
  const int b0 = own.c0, nb = own.nc, wd = b0 >> 6, sh = b0 & 63;
  unsigned long long bits = s.ok[wd] >> sh;
  if (sh) bits |= s.ok[wd + 1] << (64 - sh);
  if (nb < 64) bits &= (1ull << nb) - 1;
  return bits ? b0 + __ffsll(bits) - 1 : -1;
}

// Step 3, after a barrier, by one wavefront: the plan. Lane j holds segment j; the panels below
// one wide segment (the cheapest, or none) and that segment are the pieces, neighbouring panels
// that keep their bins one piece. `most`: a group of more rows keeps the mixed-precision loop over its bins
// (float64_most).
__device__ inline void band_plan(const BandPre& own, const double* slopes_s, int most, int nchunk, int lane, BandLds& s) {
  const int2* rows_s = reinterpret_cast<const int2*>(slopes_s);
  static_assert(MAXPANEL <= 16, "sums_16");
  const int ns = __builtin_amdgcn_readfirstlane(own.nseg), np = __builtin_amdgcn_readfirstlane(own.npanel);
  int rows = 0, row0 = 0, cand = -1, first = 0;
  if (lane < ns) {
    cand = band_of_segment(own, lane, s);
    first = own.first;
    rows = own.bins;
    row0 = own.k0;
    if (cand >= 0) {
      const int2 b = rows_s[cand];
      row0 = b.x;
      rows = b.y;
    }
  }
  // rows of the panels up to each panel, and the cheapest wide segment (0: none)
  const int pre = sums_16(lane < np ? rows : 0), excl = lane_up(pre);
  int all = __builtin_amdgcn_readlane(pre, np - 1), wide = 0;
  for (int j = np; j < ns; ++j) {
    const int n = __builtin_amdgcn_readlane(excl, __builtin_amdgcn_readlane(first, j)) + __builtin_amdgcn_readlane(rows, j);
    if (__builtin_amdgcn_readlane(cand, j) >= 0 && n < all) {
      all = n;
      wide = j;
    }
  }
  const int nf = wide ? __builtin_amdgcn_readlane(first, wide) : np;            // panels that stay
  const int wrows = __builtin_amdgcn_readlane(rows, wide), wrow0 = __builtin_amdgcn_readlane(row0, wide),
            wcand = __builtin_amdgcn_readlane(cand, wide);
  if (wide && lane == nf) {
    rows = wrows;
    row0 = wrow0;
    cand = wcand;
  }
  const int n = nf + (wide ? 1 : 0);
  const unsigned long long dir = __ballot(lane < n && cand < 0);
  const bool head = lane < n && !(cand < 0 && lane > 0 && ((dir >> (lane - 1)) & 1));
  const unsigned long long heads = __ballot(head);
  const unsigned long long after = lane < 63 ? heads >> (lane + 1) : 0;
  const int next = after ? lane + __ffsll(after) : n;        // the next piece's lane
  const int last = next - 1;
  const int lrow0 = __shfl(row0, last & 63), lrows = __shfl(rows, last & 63);
  if (head) {
    const int idx = __popcll(heads & ((1ull << lane) - 1));
    s.plan[4 + 3 * idx] = row0;
    s.plan[5 + 3 * idx] = cand < 0 ? lrow0 + lrows - row0 : rows;
    s.plan[6 + 3 * idx] = cand;
  }
  if (lane == 0) {
    const bool f64 = all <= most;
    s.plan[0] = all;
    s.plan[1] = (int)__popcll(heads);
    s.plan[2] = f64 ? 1 : 0;
    s.plan[3] = (all + nchunk - 1) / nchunk;
  }
}

// Step 3 on a calibrated event, whose segments are the calibration's node intervals: the plan keeps
// the intervals apart, from plan[4 + 2 j] each interval's first row and its rows.
__device__ inline void band_plan_cal(const BandPre& own, const double* slopes_s, int64_t M, int most, int nchunk,
                                     int lane, BandLds& s) {
  const int cand = band_of_segment(own, lane, s);
  int rows = 0;
  if (lane < own.nseg) {
    const int2 b = cand < 0 ? make_int2(own.k0, own.bins) : reinterpret_cast<const int2*>(slopes_s)[cand];
    rows = b.y;
    s.plan[4 + 2 * lane] = b.x;
    s.plan[5 + 2 * lane] = rows;
  }
  static_assert(MAXNODE - 1 <= 16, "sums_16");
  const int all = __builtin_amdgcn_readlane(sums_16(rows), 15);
  if (lane == 0) {
    const bool f64 = all <= most;
    s.plan[0] = all;
    s.plan[2] = f64 ? 1 : 0;
    s.plan[3] = ((f64 ? all : (int)M) + nchunk - 1) / nchunk;
  }
}

// Rows [q0, q1) of a group's pieces in order: fn(first row, end row, spacing). `get` reads the plan.
template <class Get, class Fn>
__device__ __forceinline__ void for_pieces(const BandHead* __restrict__ bh, double grid_step, int q0, int q1, Get get,
                                           Fn fn) {
  const int np = get(1);
  int base = 0;
  for (int i = 0; i < np && base < q1; ++i) {
    const int row0 = get(4 + 3 * i), rows = get(5 + 3 * i), cand = get(6 + 3 * i);
    const int lo = q0 > base ? q0 - base : 0, hi = q1 - base < rows ? q1 - base : rows;
    if (lo < hi) fn(row0 + lo, row0 + hi, cand < 0 ? grid_step : bh->cand[cand].step);
    base += rows;
  }
}

}  // namespace gwl
