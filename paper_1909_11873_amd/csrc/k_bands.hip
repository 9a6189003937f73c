// Building an event's band-limited rows (gwl_bands.h): which panels, segments and bands, on the
// host, and the rows' data sums on the device.
#include <hip/hip_runtime.h>

#include <math.h>
#include <string.h>

#include <algorithm>
#include <vector>

#include "gwl_bands.h"
#include "gwl_common.h"
#include "gwl_device.h"
#include "gwl_launch.h"

namespace gwl {

namespace {

constexpr double kPanelRatio = 1.5;   // of a panel's ends: t(f) of a chirp changes by 2 to 3 across one
constexpr int kWide = 4;              // wide segments (from one of the last panels to the top)
constexpr int kMinBins = 64;          // of a panel: no row set is shorter than about 50 rows
// Bands off the centre, for groups that hold a part of the arrival times (launch_order's, or a narrow
// prior's): half-widths of 32 to 91 ms, up to 0.13 s from zero and further on the side of earlier times
// by half the longest chirp, 0.7 half-widths apart (half a half-width: 1 % fewer rows with a seventh more
// bands to choose from)
constexpr double kSideTb0 = 0.032, kSideTb1 = 0.1, kSideReach = 0.13, kSideStep = 0.7;
constexpr double kTbMin = 6.371e6 / kC;  // narrowest band: detectors' arrival times alone differ by +-R/c
constexpr int64_t kMaxGrid = (int64_t)1 << 26;

// window width (nodes) at oversampling sigma, from Kaiser's estimate for 300 dB
int window_nodes(double sigma) { return (int)ceil(292.0 / (2.285 * 2.0 * M_PI * (1.0 - 1.0 / sigma))); }

// g_m'(f)
void basis_slopes(double f, double (&g)[NBASIS]) {
  const double x = cbrt(f), lf = log(f);
  g[0] = -5.0 / 3.0 / (f * f * x * x);
  g[1] = -1.0 / (f * f);
  g[2] = -2.0 / 3.0 / (f * x * x);
  g[3] = -1.0 / 3.0 / (f * x);
  g[4] = 1.0 / f;
  g[5] = 1.0 / 3.0 / (x * x);
  g[6] = (lf / 3.0 + 1.0) / (x * x);
  g[7] = 2.0 / 3.0 / x;
}

// Lowest chirp mass (solar masses) and largest arrival time (s) that a level holds: black-hole and
// neutron-star binaries near the data's time origin, and black holes that arrive within half a second. `late`:
// heavy systems with aligned spins arrive up to late f^(-2/3) after that (s, f in Hz; masses of 10 to 60, spins to
// 0.9: 0.12 s at 66 Hz, 0.02 at 1,160). A group walks every level that one of its points needs, and one that walks two
// can be the last of a launch (19,000 points of which one in 8,192 needed the second: 101 us for 53), so a level is
// to hold all of a prior (the first: all of 300,000 draws with |t_c| to 0.1 s on six grids), and few levels are better than
// many. `share` is the most that a level's rows may be of the bins. The last one is for long segments: 8,192 points
// of which 40 % are live, three detectors, 8 s (rows 0.26 of the bins), without it and with it: t_c within 0.5 s
// 148 and 86 us, all over the segment 147 and 201 (104 on every bin). `strict`: a level that takes only the
// times it is for and not the bands' margins, into which heavy systems just beyond the first level would draw their
// groups on the way to the bins (all over the segment 170).
constexpr struct { double mc, t, late, share; bool strict; } kLevels[MAXLEV] = {
    {10.0, 0.13, 1.6, 0.9, false}, {1.0, 0.13, 1.6, 0.9, true}, {10.0, 0.53, 0.0, 0.125, false}};

// The levels of an event whose bands are in `head`, bins `step` apart.
void plan_levels(BandHead& h, int64_t M, double step) {
  h.nlev[0] = h.nlev[1] = 0;
  BandLevel& every = h.lev[MAXLEV];
  every.np = 1;
  every.rows = every.n[0] = (int)M;
  every.step[0] = step;
  for (const auto& want : kLevels) {
    BandLevel v;
    memset(&v, 0, sizeof v);
    // the lowest t(f) on an interval: the Newtonian chirp's, 8 % longer, at its lower end
    const double chirp = 1.08 * 5.0 / 256.0 * pow(want.mc * kTsun, -5.0 / 3.0) * pow(M_PI, -8.0 / 3.0) * 0.6;
    auto late = [&](int i) { return want.late * 2.25 * h.gp[i][7] * h.gp[i][7]; };   // (g_7' = 2/3 f^(-1/3))
    for (int i = 0; i < MAXBRK; ++i) {
      v.lim[i].x = want.strict && i < h.nbrk ? chirp * h.gp[i][0] - want.t : -HUGE_VAL;
      v.lim[i].y = want.strict && i < h.nbrk ? want.t + late(i) : HUGE_VAL;
    }
    int band[MAXSEG], rows[MAXSEG];
    for (int s = 0; s < h.nseg; ++s) {
      band[s] = -1;
      rows[s] = h.bins[s];
      for (int c = h.c0[s]; c < h.c0[s + 1] && band[s] < 0; ++c) {
        const BandCand& b = h.cand[c];
        const double lim = BAND_FILL * b.tb;
        if (want.t + late(b.i0) - b.t0 <= lim && b.t0 + want.t - chirp * h.gp[b.i0][0] <= lim) band[s] = c, rows[s] = b.rows;
      }
    }
    // the panels below the cheapest wide segment (or all of them), and that segment
    int below = 0, best = 0, wide = -1;
    for (int p = 0; p < h.npanel; ++p) best += rows[p];
    for (int p = 0; p < h.npanel; below += rows[p++])
      for (int s = h.npanel; s < h.nseg; ++s)
        if (h.first[s] == p && band[s] >= 0 && below + rows[s] < best) best = below + rows[s], wide = s;
    const int stay = wide < 0 ? h.npanel : h.first[wide];
    for (int j = 0; j < stay + (wide < 0 ? 0 : 1); ++j) {
      const int s = j < stay ? j : wide, c = band[s];
      if (c < 0 && j > 0 && band[j - 1] < 0) {                 // neighbouring panels' bins
        v.n[v.np - 1] += rows[s];
        continue;
      }
      v.row0[v.np] = c < 0 ? h.k0[s] : h.cand[c].row0;
      v.n[v.np] = rows[s];
      v.step[v.np++] = c < 0 ? step : h.cand[c].step;
      if (c < 0) continue;
      const BandCand& b = h.cand[c];
      for (int i = b.i0; i <= b.i1; ++i) {
        v.lim[i].x = std::max(v.lim[i].x, b.t0 - BAND_FILL * b.tb);
        v.lim[i].y = std::min(v.lim[i].y, b.t0 + BAND_FILL * b.tb);
      }
    }
    v.rows = best;
    if (best > want.share * (double)M) continue;
    int n = h.nlev[0]++;
    for (; n > 0 && h.lev[n - 1].rows > best; --n) h.lev[n] = h.lev[n - 1];
    h.lev[n] = v;
  }
  while (h.nlev[1] < h.nlev[0] && h.lev[h.nlev[1]].rows <= float64_most(true, false, false, M)) ++h.nlev[1];
}

}  // namespace

// The bands of a strictly increasing grid (head.ncand = 0 when there is nothing to gain). Rows are
// numbered from `row_base`. Uniform grids space a band's rows by a multiple of half a bin, so
// that the kernel's values depend on an index difference only.
//
// `nodes`, when given, are the first bins of segments that rows may not be shared across (the last
// element is M): the calibration's node intervals, on each of which the model's factor is one cubic. The
// rows' frequencies then stay within cal_reach node spacings of the interval's ends, where that cubic is tame.
void plan_bands(const std::vector<double>& f, bool uniform, double step, int64_t row_base,
                const std::vector<int64_t>& nodes, BandHead& head, std::vector<BandGen>& gen, int64_t& nrows,
                int64_t& kvals) {
  memset(&head, 0, sizeof head);
  gen.clear();
  nrows = kvals = 0;
  const int64_t M = (int64_t)f.size();
  if (M < 2 * kMinBins || M > kMaxGrid) return;
  if (!(f.front() > 0.0) || !isfinite(f.back())) return;
  int rising = 1;                                              // (with which all are positive and finite)
  for (size_t k = 1; k < f.size(); ++k) rising &= f[k] > f[k - 1];
  if (!rising) return;
  const double flo = f.front(), fhi = f.back();
  // panels: ends in a geometric sequence, each at least kMinBins bins
  const int P = std::min(MAXPANEL, std::max(1, (int)ceil(log(fhi / flo) / log(kPanelRatio) - 1e-9)));
  std::vector<int64_t> ends{0};
  for (int i = 1; i < P; ++i) {
    const int64_t k = std::lower_bound(f.begin(), f.end(), flo * pow(fhi / flo, (double)i / P)) - f.begin();
    if (k - ends.back() >= kMinBins && M - k >= kMinBins) ends.push_back(k);
  }
  ends.push_back(M);
  if (!nodes.empty()) ends = nodes;
  const int np = (int)ends.size() - 1;
  const double hx = log(fhi / flo) / np, reach = nodes.empty() ? 0.0 : exp(cal_reach(hx) * hx);
  if (np > MAXSEG) return;
  head.npanel = np;
  struct Cand {
    BandGen g;
    BandCand c;
    double f0, f1;
  };
  std::vector<std::vector<Cand>> segs;
  bool side = true;
  auto add_segment = [&](int p) {                              // from panel p: itself, or to the top
    const bool wide = (int)segs.size() >= np;
    const int64_t ka = ends[p], kb = wide ? M : ends[p + 1], nb = kb - ka;
    const int s = (int)segs.size();
    head.first[s] = p;
    head.k0[s] = (int)ka;
    head.bins[s] = (int)nb;
    std::vector<Cand> list;
    if (nb < kMinBins) {                                       // (node intervals may be short, or empty)
      segs.push_back(list);
      return;
    }
    const double fa = f[(size_t)ka], flow = nodes.empty() ? 0.5 * fa : fa / reach;
    const double fhigh = nodes.empty() ? HUGE_VAL : reach * f[(size_t)kb - 1];
    const double width = f[(size_t)kb - 1] - fa, df = uniform ? step : width / (double)(nb - 1);
    // the band of the fewest rows centred at t0 with half-width tb or a little more, of sources from
    // fs over ws (c.rows = 0: none)
    auto band = [&](double t0, double tb, double fs, double ws) {
      Cand best;
      best.c.rows = 0;
      for (const double sigma : {1.25, 1.4, 1.6, 2.0, 2.5, 3.0}) {
        const int w = window_nodes(sigma);
        const double halves = floor(1.0 / (sigma * tb * df));
        if (halves < 3.0 || halves > 1e8) continue;             // closer than 1.5 bins
        const int half = (int)halves;
        const double h = 0.5 * half * df;
        const double rows_d = ceil(ws / h) + 2 * (w / 2) + 1, f0 = fs - (w / 2) * h;
        if (f0 < flow || f0 + rows_d * h > fhigh || rows_d > 0.8 * (double)nb) continue;
        const int rows = (int)rows_d;
        if (best.c.rows && rows >= best.c.rows) continue;
        best.c.rows = rows;
        best.c.step = h;
        best.c.tb = 0.5 / (sigma * h);
        best.c.t0 = t0;
        best.f0 = f0;
        best.f1 = f0 + (rows - 1) * h;
        best.g.src0 = (int)ka;
        best.g.nsrc = (int)nb;
        best.g.src_half = 2;
        best.g.half = half;
        best.g.n0 = -(w / 2);
        best.g.w = w;
        best.g.h = h;
        best.g.fa = fs;
        best.g.t0 = t0;
        best.g.beta = 0.98 * M_PI * 0.5 * w * (1.0 - 1.0 / sigma);
        best.g.hdf = 0.5 * df;
      }
      return best;
    };
    // Newtonian time before coalescence at fa of a chirp mass of one solar mass: the bands reach
    // 1.6 times as far (half a second at least), centred at zero and, on panels where chirps are
    // long, on their side (t0 = -0.8 tb: from coalescence to the longest; -3 tb: a factor of two)
    const double tau = 5.0 / 256.0 * pow(kTsun, -5.0 / 3.0) * pow(M_PI * fa, -8.0 / 3.0);
    const double grow = wide || tau < 0.3 ? exp2(0.25) : exp2(0.5), far = std::max(wide ? 0.36 : 0.5, 1.6 * tau);
    std::vector<std::pair<double, double>> want;               // (t0, tb)
    for (double tb = kTbMin; tb < far * grow; tb *= grow) want.push_back({0.0, tb});
    if (!wide && tau >= 0.3)
      for (const double m : {0.8, 3.0}) {
        const double lim = 1.6 * tau / (1.0 + m);
        for (double tb = lim / 6.0; tb < lim * grow; tb *= grow) want.push_back({-m * tb, tb});
      }
    // off the centre: the wide segments and the node intervals, where chirps of ten solar masses are short
    const double tau10 = tau * pow(10.0, -5.0 / 3.0);
    if (side && (wide || !nodes.empty()) && tau10 < 2.0)
      for (double tb = kSideTb0; tb < kSideTb1; tb *= exp2(0.5))
        for (int k = 1; k * kSideStep * tb <= kSideReach + 0.5 * std::min(tau10, 0.3); ++k)
          for (const int sign : {1, -1})
            if (sign < 0 || k * kSideStep * tb <= kSideReach) want.push_back({sign * k * kSideStep * tb, tb});
    // the widest band around zero comes from the bins; where it has far fewer rows than bins the others
    // are summed from its rows, which is far less work (its error adds to theirs: about 1e-14)
    Cand root;
    root.c.rows = 0;
    for (const auto& x : want) {
      if (x.first != 0.0) continue;
      const Cand c = band(0.0, x.second, fa, width);
      if (c.c.rows && (!root.c.rows || c.c.tb > root.c.tb)) root = c;
    }
    const bool staged = root.c.rows && nb >= 3 * (int64_t)root.c.rows;
    if (staged) list.push_back(root);
    for (const auto& x : want) {
      Cand c = staged ? band(x.first, x.second, root.f0, root.f1 - root.f0) : band(x.first, x.second, fa, width);
      if (!c.c.rows) continue;
      if (staged) {
        if (c.c.rows >= root.c.rows || fabs(x.first) + c.c.tb > BAND_FILL * root.c.tb) continue;
        c.g.src0 = -1;                                         // the root's rows, numbered below
        c.g.nsrc = root.c.rows;
        c.g.src_half = root.g.half;
      }
      list.push_back(c);
    }
    // fewest rows first, without those that another of no more rows holds
    std::stable_sort(list.begin(), list.end(), [](const Cand& a, const Cand& b) { return a.c.rows < b.c.rows; });
    size_t root_at = list.size();
    for (size_t i = 0; i < list.size() && staged; ++i)
      if (list[i].c.rows == root.c.rows && list[i].g.src0 >= 0) root_at = i;
    std::vector<Cand> keep;
    for (size_t i = 0; i < list.size(); ++i) {
      bool held = false;
      for (size_t j = 0; j < list.size() && !held; ++j) {
        if (i == j) continue;
        const BandCand &a = list[i].c, &b = list[j].c;
        const bool in = b.t0 - b.tb <= a.t0 - a.tb && b.t0 + b.tb >= a.t0 + a.tb;
        const bool same = a.rows == b.rows && a.t0 == b.t0 && a.tb == b.tb;
        held = in && (same ? j < i : (b.rows < a.rows || (b.rows == a.rows && j < i))) && list[j].f0 >= list[i].f0;
      }
      if (staged && i == root_at) held = false;
      if (!held && (keep.size() < 60 || i == root_at)) keep.push_back(list[i]);
    }
    segs.push_back(keep);
  };
  auto add_segments = [&] {
    segs.clear();
    for (int p = 0; p < np; ++p) add_segment(p);
    for (int p = std::max(0, np - 1 - kWide); p < np - 1 && nodes.empty(); ++p) add_segment(p);
  };
  add_segments();
  size_t all = 0;
  for (const auto& l : segs) all += l.size();
  if (all > MAXCAND) {
    side = false;
    add_segments();
  }
  head.nseg = (int)segs.size();
  // the intervals on which t(f) is bounded, over every frequency that a row has
  double f0 = flo, f1 = fhi;
  int ncand = 0;
  for (auto& l : segs) {
    if (ncand + (int)l.size() > MAXCAND) l.clear();            // (60 bands at most of 18 segments: not on real grids)
    ncand += (int)l.size();
    for (const Cand& c : l) {
      f0 = std::min(f0, c.f0);
      f1 = std::max(f1, c.f1);
    }
  }
  // (the slope of f^(1/3) ln f turns at exp(-3/2) Hz, and an interval's slopes have to be monotone)
  if (ncand == 0 || f0 < 0.25) {
    head.npanel = head.nseg = 0;
    return;
  }
  const int nbrk = std::min(MAXBRK, std::max(1, (int)ceil(log(f1 / f0) / log(1.15))));
  head.nbrk = nbrk;
  const double lr = log(f1 / f0) / nbrk;
  for (int i = 0; i <= nbrk; ++i) basis_slopes(f0 * exp(lr * i), head.gp[i]);
  int c = 0;
  for (int s = 0; s < head.nseg; ++s) {
    head.c0[s] = c;
    for (Cand& x : segs[s]) {
      x.c.i0 = std::min(nbrk - 1, std::max(0, (int)floor(log(x.f0 / f0) / lr - 1e-9)));
      x.c.i1 = std::min(nbrk - 1, std::max(0, (int)floor(log(x.f1 / f0) / lr + 1e-9)));
      x.c.row0 = (int)(row_base + nrows);
      x.g.row0 = x.c.row0;
      x.g.rows = x.c.rows;
      x.g.klen = uniform && x.g.src0 >= 0 ? (x.g.w * x.g.half) / 2 + 1 : 0;
      x.g.koff = kvals;
      kvals += x.g.klen;
      nrows += x.c.rows;
      head.cand[c++] = x.c;
      gen.push_back(x.g);
    }
  }
  head.c0[head.nseg] = c;
  head.ncand = c;
  // the staged bands' sources
  for (int s = 0; s < head.nseg; ++s)
    for (int i = head.c0[s]; i < head.c0[s + 1]; ++i)
      if (gen[i].src0 >= 0)
        for (int j = head.c0[s]; j < head.c0[s + 1]; ++j)
          if (gen[j].src0 == -1 && gen[j].nsrc == gen[i].rows) gen[j].src0 = -2 - gen[i].row0;
  for (BandGen& g : gen)
    if (g.src0 < -1) g.src0 = -2 - g.src0;
  if (nodes.empty()) plan_levels(head, M, step);
}

// K(x) exp(-2 pi i t0 d) at x nodes, d Hz from a row (d >= 0; conjugate below)
__device__ inline double2 band_kernel(const BandGen& g, double x, double d) {
  const double z = 2.0 * x / (double)g.w, r2 = 1.0 - z * z;
  if (!(r2 > 0.0)) return make_double2(0.0, 0.0);
  const double sc = x != 0.0 ? sinpi(x) / (kPi * x) : 1.0;
  const double v = sc * exp(g.beta * (sqrt(r2) - 1.0));
  double sn, cs;
  sincos_cycles_f64(g.t0 * d, sn, cs);
  return make_double2(v * cs, -v * sn);
}

// kernel values of a uniform grid's bands, by half-bin distance
__global__ __launch_bounds__(256) void k_band_kernel(const BandGen* __restrict__ gen, double2* __restrict__ kv) {
  const BandGen g = gen[blockIdx.y];
  for (int j = blockIdx.x * 256 + threadIdx.x; j < g.klen; j += gridDim.x * 256)
    kv[g.koff + j] = band_kernel(g, (double)j / (double)g.half, (double)j * g.hdf);
}

// The rows: one wavefront per four neighbouring rows of a band, its lanes over the sources within
// their windows (each source is read once for the four rows). Bound by L2 reads of the sources; 8 s, three
// detectors, 118,000 rows: 369 us in the two launches; 128 s: 779 (9.9 ms when every band was summed from
// the bins).
constexpr int BR_ROWS = 4;
constexpr int BR_WAVES = 4;
template <int ND>
__global__ __launch_bounds__(BR_WAVES * WAVE) void k_band_rows(const BandGen* __restrict__ gen,
                                                               const int2* __restrict__ blk, bool uniform,
                                                               const double2* __restrict__ kv, RowF64<ND>* tab,
                                                               RowGradF64* __restrict__ gtab) {
  const int2 b = blk[blockIdx.x];
  const BandGen g = gen[b.x];
  const int w = (int)(threadIdx.x / WAVE), lane = (int)(threadIdx.x % WAVE);
  const int q = b.y + w * BR_ROWS;
  if (q >= g.rows) return;
  // sources of the four windows together
  int klo, khi;
  const double fq0 = g.fa + (double)(g.n0 + q) * g.h;
  // bins of a grid that is not uniform are looked up by frequency; all else lies on multiples of half a bin
  const bool lattice = uniform || g.src_half != 2;
  if (lattice) {
    const int64_t reach = (int64_t)g.w * g.half / 2 + g.src_half, at = (int64_t)g.half * (g.n0 + q);
    const int64_t lo = (at - reach) / g.src_half - 1, hi = (at + (int64_t)g.half * (BR_ROWS - 1) + reach) / g.src_half + 2;
    klo = (int)(lo < 0 ? 0 : (lo > g.nsrc ? g.nsrc : lo));
    khi = (int)(hi < 0 ? 0 : (hi > g.nsrc ? g.nsrc : hi));
  } else {
    auto first_at = [&](double x) {                    // first source at or above x
      int lo = 0, hi = g.nsrc;
      while (lo < hi) {
        const int mid = (lo + hi) / 2;
        if (tab[g.src0 + mid].f < x) lo = mid + 1;
        else hi = mid;
      }
      return lo;
    };
    klo = first_at(fq0 - 0.5 * g.w * g.h);
    khi = first_at(fq0 + (0.5 * g.w + (BR_ROWS - 1)) * g.h);
  }
  double acc[BR_ROWS][2 * ND];
#pragma unroll
  for (int j = 0; j < BR_ROWS; ++j)
#pragma unroll
    for (int z = 0; z < 2 * ND; ++z) acc[j][z] = 0.0;
  for (int k = klo + lane; k < khi; k += WAVE) {
    double u[2 * ND];
#pragma unroll
    for (int z = 0; z < 2 * ND; ++z) u[z] = tab[g.src0 + k].u[z];
#pragma unroll
    for (int j = 0; j < BR_ROWS; ++j) {
      double2 kk;
      bool neg;
      if (lattice) {
        const int64_t d = (int64_t)g.src_half * k - (int64_t)g.half * (g.n0 + q + j);
        const int64_t ad = d < 0 ? -d : d;
        if (g.klen > 0) kk = ad < g.klen ? kv[g.koff + ad] : make_double2(0.0, 0.0);
        else kk = band_kernel(g, (double)ad / (double)g.half, (double)ad * g.hdf);
        neg = d < 0;
      } else {
        const double d = tab[g.src0 + k].f - (fq0 + j * g.h), ad = fabs(d);
        kk = band_kernel(g, ad / g.h, ad);
        neg = d < 0.0;
      }
      const double ki = neg ? -kk.y : kk.y;
#pragma unroll
      for (int d = 0; d < ND; ++d) {
        acc[j][2 * d] = fma(u[2 * d], kk.x, fma(-u[2 * d + 1], ki, acc[j][2 * d]));
        acc[j][2 * d + 1] = fma(u[2 * d], ki, fma(u[2 * d + 1], kk.x, acc[j][2 * d + 1]));
      }
    }
  }
#pragma unroll
  for (int j = 0; j < BR_ROWS; ++j)
#pragma unroll
    for (int z = 0; z < 2 * ND; ++z)
#pragma unroll
      for (int off = WAVE / 2; off > 0; off >>= 1) acc[j][z] += __shfl_xor(acc[j][z], off);
#pragma unroll
  for (int j = 0; j < BR_ROWS; ++j) {
    if (lane != j || q + j >= g.rows) continue;
    const double f = g.fa + (double)(g.n0 + q + j) * g.h;
    RowF64<ND> row;
    const double x = cbrt(f), w2 = 1.0 / f, lnf = log(f);
    row.f = f; row.x = x; row.w = w2 / (x * x); row.w2 = w2; row.lnf = lnf;
#pragma unroll
    for (int z = 0; z < 2 * ND; ++z) row.u[z] = acc[j][z];
    tab[g.row0 + q + j] = row;
    RowGradF64 gd;
    gd.g2 = w2 * x; gd.g3 = w2 * x * x; gd.g6 = x * lnf; gd.g7 = x * x;
    gtab[g.row0 + q + j] = gd;
  }
}

// The workgroups' rows (band, first row): the bands made from bins first (nblk[0] workgroups), then
// those made from their rows (nblk[1]).
void band_blocks(const std::vector<BandGen>& gen, int64_t M, std::vector<int2>& blk, int (&nblk)[2]) {
  blk.clear();
  for (int stage = 0; stage < 2; ++stage) {
    const size_t at = blk.size();
    for (size_t c = 0; c < gen.size(); ++c)
      if ((gen[c].src0 >= M) == (stage == 1))
        for (int q = 0; q < gen[c].rows; q += BR_WAVES * BR_ROWS) blk.push_back(make_int2((int)c, q));
    nblk[stage] = (int)(blk.size() - at);
  }
}

template <int ND>
static hipError_t bands_nd(bool uniform, const BandGen* gen, int ncand, const int2* blk, const int (&nblk)[2], double2* kv,
                           void* tab, RowGradF64* gtab, hipStream_t s) {
  if (uniform) hipLaunchKernelGGL(k_band_kernel, dim3(8, (unsigned)ncand), dim3(256), 0, s, gen, kv);
  for (int stage = 0; stage < 2; ++stage) {
    if (nblk[stage] > 0)
      hipLaunchKernelGGL(k_band_rows<ND>, dim3((unsigned)nblk[stage]), dim3(BR_WAVES * WAVE), 0, s, gen, blk, uniform,
                         (const double2*)kv, (RowF64<ND>*)tab, gtab);
    blk += nblk[stage];
  }
  return hipGetLastError();
}

hipError_t launch_bands(int nd, bool uniform, const BandGen* gen, int ncand, const int2* blk, const int (&nblk)[2],
                        double2* kv, void* tab, RowGradF64* gtab, hipStream_t s) {
  if (ncand < 1 || nblk[0] < 1 || nblk[1] < 0 || !gen || !blk) return hipErrorInvalidValue;
  switch (nd) {
    case 1: return bands_nd<1>(uniform, gen, ncand, blk, nblk, kv, tab, gtab, s);
    case 2: return bands_nd<2>(uniform, gen, ncand, blk, nblk, kv, tab, gtab, s);
    case 3: return bands_nd<3>(uniform, gen, ncand, blk, nblk, kv, tab, gtab, s);
    case 4: return bands_nd<4>(uniform, gen, ncand, blk, nblk, kv, tab, gtab, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace gwl
