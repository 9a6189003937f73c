// Host runtime of the C ABI in include/gwlike.h: argument checking, event tables, workspace,
// launch sequencing, tile choice. All computation happens in the kernels.
#include <hip/hip_runtime.h>

#include <limits.h>
#include <math.h>
#include <stdarg.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <mutex>
#include <string>
#include <utility>
#include <vector>

#include "../../include/gwlike.h"
#include "gwl_bands.h"
#include "gwl_common.h"
#include "gwl_device.h"
#include "gwl_launch.h"
#include "gwl_runtime.h"

using namespace gwl;

namespace gwl {

static thread_local std::string g_err;

gwl_status fail(gwl_status st, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  g_err = buf;
  return st;
}

// The error is the caller's from here on: it is taken out of the runtime's own record, which the launch
// wrappers read back, so that a call after it (an entry point's retry in less memory, or the next one) does not report it again.
gwl_status hip_fail(hipError_t e, const char* what) {
  (void)hipGetLastError();
  if (e == hipErrorOutOfMemory) return fail(GWL_E_NOMEM, "%s: %s", what, hipGetErrorString(e));
  return fail(GWL_E_DEVICE, "%s: %s", what, hipGetErrorString(e));
}

void clear_error() { g_err.clear(); }

size_t row64_bytes(int nd) { return 40 + 16 * (size_t)nd; }
size_t row32_bytes(int nd) { return 40 + 8 * (size_t)nd; }

// Detector tensor and vertex of an L-shaped detector (arms horizontal, azimuths clockwise
// from North) on a spherical Earth.
static void detector_geometry(const gwl_detector& d, double dt[6], double r[3]) {
  const double RE = 6.371e6;
  const double sl = sin(d.lat), cl = cos(d.lat), so = sin(d.lon), co = cos(d.lon);
  const double north[3] = {-sl * co, -sl * so, cl};
  const double east[3] = {-so, co, 0.0};
  double xa[3], ya[3];
  for (int i = 0; i < 3; ++i) {
    xa[i] = cos(d.xarm_az) * north[i] + sin(d.xarm_az) * east[i];
    ya[i] = cos(d.yarm_az) * north[i] + sin(d.yarm_az) * east[i];
  }
  const int ii[6] = {0, 1, 2, 0, 0, 1}, jj[6] = {0, 1, 2, 1, 2, 2};
  for (int m = 0; m < 6; ++m) dt[m] = 0.5 * (xa[ii[m]] * xa[jj[m]] - ya[ii[m]] * ya[jj[m]]);
  r[0] = RE * cl * co;
  r[1] = RE * cl * so;
  r[2] = RE * sl;
}

gwl_status make_geom(const gwl_detector* dets, int ndet, double gmst, EventGeom& g) {
  if (!dets) return fail(GWL_E_INVALID, "dets is null");
  if (ndet < 1 || ndet > GWL_MAX_DET) return fail(GWL_E_SHAPE, "ndet=%d outside [1, %d]", ndet, GWL_MAX_DET);
  if (!isfinite(gmst)) return fail(GWL_E_INVALID, "gmst is not finite");
  memset(&g, 0, sizeof g);
  g.ndet = ndet;
  g.gmst = gmst;
  for (int d = 0; d < ndet; ++d) {
    const gwl_detector& x = dets[d];
    if (!isfinite(x.lat) || !isfinite(x.lon) || !isfinite(x.xarm_az) || !isfinite(x.yarm_az))
      return fail(GWL_E_INVALID, "detector %d has a non-finite angle", d);
    detector_geometry(x, g.dt[d], g.r[d]);
  }
  return GWL_OK;
}

gwl_status check_device(int dev) {
  int cur = -1;
  hipError_t e = hipGetDevice(&cur);
  if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
  if (cur != dev) return fail(GWL_E_INVALID, "event lives on device %d but device %d is current", dev, cur);
  return GWL_OK;
}

}  // namespace gwl

namespace gwl {

// A grid is uniform when every step f_{k+1} - f_k equals the mean step (f_{M-1} - f_0) / (M - 1)
// to within 8 ulp of the highest frequency: a grid built as f_0 + k df in float64 is uniform.
static bool grid_is_uniform(const std::vector<double>& f, double& step) {
  const size_t M = f.size();
  step = M > 1 ? (f[M - 1] - f[0]) / (double)(M - 1) : 1.0;
  const double tol = 8.0 * ldexp(fabs(f[M - 1]), -52);
  for (size_t k = 0; k + 1 < M; ++k)
    if (!(fabs((f[k + 1] - f[k]) - step) <= tol)) return false;
  return true;
}

// Tables of the optional ISCO cut-off, built on the host in float64 (once per event): the grid
// (which must increase) and per detector the running sums Kc[k] = sum_{j < k} 4 df f_j^(-7/3) / S_j,
// k = 0..M, so that <h|h> of a point cut after its first kc bins is A^2 |Q_det|^2 Kc[kc].
static gwl_status isco_tables(gwl_event ev, const double* fgrid, const double* psd, hipStream_t s) {
  const int64_t M = ev->M;
  const int nd = ev->ndet;
  std::vector<double> f((size_t)M), ps((size_t)M * nd);
  hipError_t e = hipMemcpyAsync(f.data(), fgrid, sizeof(double) * M, hipMemcpyDeviceToHost, s);
  if (e == hipSuccess) e = hipMemcpyAsync(ps.data(), psd, sizeof(double) * M * nd, hipMemcpyDeviceToHost, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  if (e != hipSuccess) return hip_fail(e, "grid read-back");
  for (int64_t k = 1; k < M; ++k)
    if (!(f[(size_t)k] > f[(size_t)k - 1]))
      return fail(GWL_E_INVALID, "the ISCO cut-off needs an increasing frequency grid (bin %lld)", (long long)k);
  std::vector<double> kc((size_t)(M + 1) * nd);
  for (int d = 0; d < nd; ++d) {
    double acc = 0.0;
    kc[(size_t)d * (M + 1)] = 0.0;
    for (int64_t k = 0; k < M; ++k) {
      acc += 4.0 * ev->df * pow(f[(size_t)k], -7.0 / 3.0) / ps[(size_t)d * M + k];
      kc[(size_t)d * (M + 1) + k + 1] = acc;
    }
  }
  e = hipMalloc((void**)&ev->fgrid, sizeof(double) * M);
  if (e == hipSuccess) e = hipMalloc((void**)&ev->kcum, sizeof(double) * kc.size());
  if (e == hipSuccess) e = hipMemcpy(ev->fgrid, f.data(), sizeof(double) * M, hipMemcpyHostToDevice);
  if (e == hipSuccess) e = hipMemcpy(ev->kcum, kc.data(), sizeof(double) * kc.size(), hipMemcpyHostToDevice);
  if (e != hipSuccess) return hip_fail(e, "ISCO tables");
  ev->ech.isco = 1;
  ev->ech.grid_df = M > 1 ? (f[(size_t)M - 1] - f[0]) / (double)(M - 1) : 1.0;
  e = hipMemcpy(ev->ec, &ev->ech, sizeof(EventConst), hipMemcpyHostToDevice);
  if (e != hipSuccess) return hip_fail(e, "ISCO tables");
  return GWL_OK;
}

}  // namespace gwl

// ------------------------------------------------------------------------------------------------
// C ABI
// ------------------------------------------------------------------------------------------------
extern "C" {

const char* gwl_last_error(void) { return g_err.c_str(); }

const char* gwl_version(void) { return "gwlike 0.1 (gfx950)"; }

}  // extern "C"

namespace gwl {

// bands: whether the event may walk band-limited rows (a relative-binning event's grid tables are
// replaced by its edges', and the ISCO cut-off walks every bin); nnode: calibration nodes per
// detector, whose intervals the rows then keep to (0: none)
static gwl_status event_create(const double* data, const double* psd, const gwl_detector* dets, int ndet,
                               const double* fgrid, int64_t M, double df, double gmst, unsigned flags, void* stream,
                               bool bands, int nnode, gwl_event* out);

// Band-limited rows of a new event whose grid rows are queued on s: the rows' tables follow the
// grid's in tab64 and g64 (allocated with room for them).
struct BandHost {
  BandHead head;
  std::vector<BandGen> gen;
  std::vector<int2> blk;
  int nblk[2] = {0, 0};
  int64_t nrows = 0, kvals = 0;
};

// One device allocation for several arrays: take() the offsets, then base + offset (an allocation, and
// the wait when it is freed, takes longer than preparing a small event's tables).
struct Slab {
  size_t bytes = 0;
  size_t take(size_t n) {
    const size_t at = bytes;
    bytes += (n + 255) / 256 * 256;
    return at;
  }
};

// First bins of the calibration's node intervals (nnode - 1 of them, equal in ln f; then M).
static void cal_intervals(const std::vector<double>& f, int nnode, std::vector<int64_t>& first) {
  const int64_t M = (int64_t)f.size();
  const double x0 = log(f.front()), h = (log(f.back()) - x0) / (nnode - 1);
  first.assign((size_t)nnode, M);
  for (int64_t k = M - 1; k >= 0; --k) {
    const double s = std::min(std::max((log(f[(size_t)k]) - x0) / h, 0.0), (double)(nnode - 1));
    first[(size_t)std::min(std::max((int)floor(s), 0), nnode - 2)] = k;
  }
  first[0] = 0;
  for (int j = nnode - 2; j >= 1; --j) first[j] = std::min(first[j], first[j + 1]);  // empty: where the next starts
}

// Rows that a point of a black-hole binary near the data's time origin walks (chirp mass ten solar
// masses, arrival within 0.125 s): what a launch's shape is chosen for.
static int64_t typical_rows(const BandHead& h, int64_t M) {
  if (h.ncand == 0) return M;
  std::vector<int64_t> rows((size_t)h.nseg);
  for (int s = 0; s < h.nseg; ++s) {
    rows[s] = h.bins[s];
    for (int c = h.c0[s]; c < h.c0[s + 1]; ++c) {
      const BandCand& b = h.cand[c];
      // -tau(f) at the lowest frequency of the band's rows, from g_0' = -5/3 f^-8/3
      const double tau = 5.0 / 256.0 * pow(10.0 * kTsun, -5.0 / 3.0) * pow(M_PI, -8.0 / 3.0) * -0.6 * h.gp[b.i0][0];
      const double lim = BAND_FILL * b.tb;
      if (0.125 - b.t0 <= lim && b.t0 + 0.125 + tau <= lim) {
        rows[s] = std::min<int64_t>(rows[s], b.rows);
        break;
      }
    }
  }
  int64_t below = 0, best = -1;
  for (int p = 0; p < h.npanel; ++p) {
    for (int s = h.npanel; s < h.nseg; ++s)
      if (h.first[s] == p && (best < 0 || below + rows[s] < best)) best = below + rows[s];
    below += rows[p];
  }
  return best < 0 ? below : std::min(best, below);
}

}  // namespace gwl

extern "C" {

gwl_status gwl_event_create(const double* data, const double* psd, const gwl_detector* dets, int ndet,
                            const double* fgrid, int64_t M, double df, double gmst, unsigned flags, void* stream,
                            gwl_event* out) {
  return event_create(data, psd, dets, ndet, fgrid, M, df, gmst, flags, stream, !(flags & GWL_F_ISCO_CUTOFF), 0, out);
}

}  // extern "C"

namespace gwl {

static gwl_status event_create(const double* data, const double* psd, const gwl_detector* dets, int ndet,
                               const double* fgrid, int64_t M, double df, double gmst, unsigned flags, void* stream,
                               bool bands, int nnode, gwl_event* out) {
  clear_error();
  if (!out) return fail(GWL_E_INVALID, "out is null");
  *out = nullptr;
  if (!data || !psd || !fgrid) return fail(GWL_E_INVALID, "data, psd and fgrid must be device pointers");
  if (M < 1 || M > (int64_t)1 << 30) return fail(GWL_E_SHAPE, "M=%lld outside [1, 2^30]", (long long)M);
  if (!(df > 0.0) || !isfinite(df)) return fail(GWL_E_INVALID, "df must be finite and positive");
  if (flags & ~(unsigned)GWL_F_ISCO_CUTOFF) return fail(GWL_E_UNSUPPORTED, "flags=0x%x: unknown flags", flags);
  EventGeom g;
  gwl_status st = make_geom(dets, ndet, gmst, g);
  if (st != GWL_OK) return st;

  gwl_event ev = new (std::nothrow) gwl_event_s();
  if (!ev) return fail(GWL_E_NOMEM, "host allocation failed");
  ev->ndet = ndet;
  ev->M = M;
  ev->df = df;
  ev->gmst = gmst;
  ev->geom = g;
  for (int d = 0; d < ndet; ++d) ev->dets[d] = dets[d];
  hipStream_t s = (hipStream_t)stream;
  hipError_t e = hipGetDevice(&ev->device);
  // the grid on the host: its step, whether the float64 loop may carry detector phasors by a fixed
  // rotation, and its bands
  std::vector<double> fh((size_t)M);
  if (e == hipSuccess) e = hipMemcpyAsync(fh.data(), fgrid, sizeof(double) * M, hipMemcpyDeviceToHost, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  if (e != hipSuccess) {
    gwl_event_destroy(ev);
    return hip_fail(e, "grid read-back");
  }
  double step = 1.0;
  const bool uniform = grid_is_uniform(fh, step);
  BandHost bh;
  memset(&bh.head, 0, sizeof bh.head);
  if (bands) {
    std::vector<int64_t> nodes;
    if (nnode > 0) cal_intervals(fh, nnode, nodes);
    plan_bands(fh, uniform, step, M + TAB_PAD, nodes, bh.head, bh.gen, bh.nrows, bh.kvals);
    band_blocks(bh.gen, M, bh.blk, bh.nblk);
    for (int sg = 0; nnode > 0 && sg < bh.head.nseg; ++sg)
      for (int c = bh.head.c0[sg]; c < bh.head.c0[sg + 1]; ++c)
        for (int q = 0; q < bh.gen[c].rows; ++q) {
          ev->band_f.push_back(bh.gen[c].fa + (double)(bh.gen[c].n0 + q) * bh.gen[c].h);
          ev->band_seg.push_back(sg);
        }
  }
  ev->M_loop = bands ? typical_rows(bh.head, M) : M;
  for (int i = 0; i < 2; ++i) ev->nlev[i] = bh.head.nlev[i];
  const int64_t rows = M + TAB_PAD + (bh.nrows > 0 ? bh.nrows + TAB_PAD : 0);
  const int nblk = prep_blocks(M);
  Slab keep, work;
  const size_t o64 = keep.take(row64_bytes(ndet) * rows), o32 = keep.take(row32_bytes(ndet) * (M + TAB_PAD));
  const size_t og32 = keep.take(sizeof(RowGradF32) * M);
  const size_t og64 = keep.take(sizeof(RowGradF64) * (bh.nrows > 0 ? rows : M));
  const size_t oec = keep.take(sizeof(EventConst)), obh = keep.take(bh.nrows > 0 ? sizeof(BandHead) : 0);
  const size_t wpart = work.take(sizeof(double) * prep_scratch_doubles(ndet, M));
  const size_t wgen = work.take(sizeof(BandGen) * bh.gen.size()), wblk = work.take(sizeof(int2) * bh.blk.size());
  const size_t wkv = work.take(sizeof(double2) * (size_t)bh.kvals);
  char *scratch = nullptr, *slab = nullptr;
  e = hipMalloc((void**)&slab, keep.bytes);
  if (e == hipSuccess) {
    ev->slab = slab;
    ev->tab64 = slab + o64;
    ev->tab32 = slab + o32;
    ev->g32 = (RowGradF32*)(slab + og32);
    ev->g64 = (RowGradF64*)(slab + og64);
    ev->ec = (EventConst*)(slab + oec);
    e = hipMalloc((void**)&scratch, work.bytes);
  }
  if (e == hipSuccess)
    e = hipMemsetAsync((char*)ev->tab64 + row64_bytes(ndet) * M, 0, row64_bytes(ndet) * TAB_PAD, s);
  if (e == hipSuccess && bh.nrows > 0)
    e = hipMemsetAsync((char*)ev->tab64 + row64_bytes(ndet) * (rows - TAB_PAD), 0, row64_bytes(ndet) * TAB_PAD, s);
  if (e == hipSuccess)
    e = hipMemsetAsync((char*)ev->tab32 + row32_bytes(ndet) * M, 0, row32_bytes(ndet) * TAB_PAD, s);
  if (e == hipSuccess)
    e = launch_prep(ndet, data, psd, fgrid, M, df, ev->tab64, ev->tab32, ev->g32, ev->g64, (double*)(scratch + wpart),
                    nblk, ev->ec, s);
  // the band-limited rows, from the grid's (after rejected inputs they are never used)
  if (e == hipSuccess && bh.nrows > 0) {
    ev->bands = (BandHead*)(slab + obh);
    e = hipMemcpyAsync(ev->bands, &bh.head, sizeof(BandHead), hipMemcpyHostToDevice, s);
    if (e == hipSuccess)
      e = hipMemcpyAsync(scratch + wgen, bh.gen.data(), sizeof(BandGen) * bh.gen.size(), hipMemcpyHostToDevice, s);
    if (e == hipSuccess)
      e = hipMemcpyAsync(scratch + wblk, bh.blk.data(), sizeof(int2) * bh.blk.size(), hipMemcpyHostToDevice, s);
    if (e == hipSuccess)
      e = launch_bands(ndet, uniform, (const BandGen*)(scratch + wgen), (int)bh.gen.size(), (const int2*)(scratch + wblk),
                       bh.nblk, (double2*)(scratch + wkv), ev->tab64, ev->g64, s);
  }
  if (e == hipSuccess) e = hipMemcpyAsync(&ev->ech, ev->ec, sizeof(EventConst), hipMemcpyDeviceToHost, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  if (e == hipSuccess) {
    ev->ech.uniform = uniform ? 1 : 0;
    ev->ech.grid_df = step;
    e = hipMemcpyAsync(ev->ec, &ev->ech, sizeof(EventConst), hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
  }
  if (scratch) (void)hipFree(scratch);
  if (e != hipSuccess) {
    gwl_event_destroy(ev);
    return hip_fail(e, "event preparation");
  }
  if (ev->ech.bad) {
    gwl_event_destroy(ev);
    return fail(GWL_E_INVALID, "rejected inputs: every PSD value and frequency must be finite and positive and "
                               "every data value finite");
  }
  if (flags & GWL_F_ISCO_CUTOFF) {
    st = isco_tables(ev, fgrid, psd, s);
    if (st != GWL_OK) {
      gwl_event_destroy(ev);
      return st;
    }
  }
  *out = ev;
  return GWL_OK;
}

}  // namespace gwl

extern "C" {

// Relative-binning edges on the grid: the bins where floor(dpsi(f) / eps) changes, plus both
// ends, with dpsi(f) = 2 pi sum_gamma sign(gamma) (f / f_gamma)^gamma over the post-Newtonian
// phase power laws gamma = -5/3, -2/3, 1, 5/3, 7/3 (f_gamma = f_hi for gamma > 0, f_lo below):
// the largest phase difference between two waveforms of the model grows no faster than dpsi.
static std::vector<int64_t> rb_edges(const std::vector<double>& f, double eps) {
  const double flo = f.front(), fhi = f.back();
  const double gam[5] = {-5.0 / 3.0, -2.0 / 3.0, 1.0, 5.0 / 3.0, 7.0 / 3.0};
  auto dpsi = [&](double x) {
    double s = 0.0;
    for (double g : gam) s += (g > 0 ? 1.0 : -1.0) * pow(x / (g > 0 ? fhi : flo), g);
    return 2.0 * M_PI * s;
  };
  std::vector<int64_t> idx{0};
  double prev = floor(dpsi(f[0]) / eps);
  for (size_t k = 1; k < f.size(); ++k) {
    const double c = floor(dpsi(f[k]) / eps);
    if (c != prev) idx.push_back((int64_t)k);
    prev = c;
  }
  if (idx.back() != (int64_t)f.size() - 1) idx.push_back((int64_t)f.size() - 1);
  return idx;
}

gwl_status gwl_event_create_rb(const double* data, const double* psd, const gwl_detector* dets, int ndet,
                               const double* fgrid, int64_t M, double df, double gmst, const double* theta_fid,
                               double eps, unsigned flags, void* stream, gwl_event* out) {
  clear_error();
  if (!out) return fail(GWL_E_INVALID, "out is null");
  *out = nullptr;
  if (!theta_fid) return fail(GWL_E_INVALID, "theta_fid must be a host array of 11 values");
  for (int i = 0; i < NPARAM; ++i)
    if (!isfinite(theta_fid[i])) return fail(GWL_E_INVALID, "theta_fid[%d] is not finite", i);
  if (!(eps > 0.0) || !isfinite(eps)) return fail(GWL_E_INVALID, "eps must be finite and positive");
  if (flags & GWL_F_ISCO_CUTOFF)
    return fail(GWL_E_UNSUPPORTED, "the ISCO cut-off is not available with relative binning");
  gwl_event ev = nullptr;
  gwl_status st = event_create(data, psd, dets, ndet, fgrid, M, df, gmst, flags, stream, false, 0, &ev);
  if (st != GWL_OK) return st;
  hipStream_t s = (hipStream_t)stream;
  // grid on the host, edges
  std::vector<double> fh((size_t)M);
  hipError_t e = hipMemcpyAsync(fh.data(), fgrid, sizeof(double) * M, hipMemcpyDeviceToHost, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  if (e != hipSuccess) {
    gwl_event_destroy(ev);
    return hip_fail(e, "grid read-back");
  }
  const std::vector<int64_t> idx = rb_edges(fh, eps);
  const int nedge = (int)idx.size();
  // fiducial coefficients through the ordinary set-up (no offsets, no gain)
  double *th = nullptr, *coef = nullptr, *w = nullptr;
  int64_t* d_idx = nullptr;
  char* slab = nullptr;
  void *tab64 = nullptr, *tab32 = nullptr;
  RowGradF32* g32 = nullptr;
  RowGradF64* g64 = nullptr;
  EventConst* ec = nullptr;
  std::vector<double> hcoef((size_t)NCOEF * WAVE);
  const int nd = ev->ndet;
  e = hipMalloc((void**)&th, sizeof(double) * NPARAM);
  if (e == hipSuccess) e = hipMalloc((void**)&coef, sizeof(double) * NCOEF * WAVE);
  if (e == hipSuccess) e = hipMemcpyAsync(th, theta_fid, sizeof(double) * NPARAM, hipMemcpyHostToDevice, s);
  if (e == hipSuccess) e = launch_setup(nd, ev->geom, nullptr, th, 1, WAVE, coef, s);
  if (e == hipSuccess)
    e = hipMemcpyAsync(hcoef.data(), coef, sizeof(double) * NCOEF * WAVE, hipMemcpyDeviceToHost, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  bool fid_ok = e == hipSuccess;
  if (fid_ok) {
    for (int m = 0; m < NBASIS; ++m) {
      ev->ech.fa[m] = hcoef[(size_t)(CO_A + m) * WAVE];
      fid_ok &= isfinite(ev->ech.fa[m]);
    }
    for (int d = 0; d < MAXDET; ++d) ev->ech.fT[d] = d < nd ? hcoef[(size_t)(CO_T + d) * WAVE] : 0.0;
    for (int d = 0; d < nd; ++d) fid_ok &= isfinite(ev->ech.fT[d]);
  }
  if (e == hipSuccess && !fid_ok) {
    (void)hipFree(th);
    (void)hipFree(coef);
    gwl_event_destroy(ev);
    return fail(GWL_E_INVALID, "theta_fid is outside the model's domain");
  }
  // edge tables (the edges are not a uniform grid)
  ev->ech.uniform = 0;
  if (e == hipSuccess) e = hipMemcpyAsync(ev->ec, &ev->ech, sizeof(EventConst), hipMemcpyHostToDevice, s);
  if (e == hipSuccess) e = hipMalloc((void**)&d_idx, sizeof(int64_t) * nedge);
  if (e == hipSuccess) e = hipMemcpyAsync(d_idx, idx.data(), sizeof(int64_t) * nedge, hipMemcpyHostToDevice, s);
  if (e == hipSuccess) e = hipMalloc((void**)&w, sizeof(double) * rb_scratch_doubles(nd, nedge));
  Slab keep;
  const size_t o64 = keep.take(row64_bytes(nd) * (nedge + TAB_PAD)), o32 = keep.take(row32_bytes(nd) * (nedge + TAB_PAD));
  const size_t og32 = keep.take(sizeof(RowGradF32) * nedge), og64 = keep.take(sizeof(RowGradF64) * nedge);
  const size_t oec = keep.take(sizeof(EventConst));
  if (e == hipSuccess) e = hipMalloc((void**)&slab, keep.bytes);
  if (e == hipSuccess) {
    tab64 = slab + o64;
    tab32 = slab + o32;
    g32 = (RowGradF32*)(slab + og32);
    g64 = (RowGradF64*)(slab + og64);
    ec = (EventConst*)(slab + oec);
    e = hipMemcpyAsync(ec, ev->ec, sizeof(EventConst), hipMemcpyDeviceToDevice, s);
  }
  if (e == hipSuccess) e = hipMemsetAsync((char*)tab64 + row64_bytes(nd) * nedge, 0, row64_bytes(nd) * TAB_PAD, s);
  if (e == hipSuccess) e = hipMemsetAsync((char*)tab32 + row32_bytes(nd) * nedge, 0, row32_bytes(nd) * TAB_PAD, s);
  if (e == hipSuccess) e = launch_rb(nd, ev->tab64, ev->g32, ev->g64, d_idx, nedge, w, ec, tab64, tab32, g32, g64, s);
  if (e == hipSuccess) e = hipMemcpyAsync(&ev->ech, ec, sizeof(EventConst), hipMemcpyDeviceToHost, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  (void)hipFree(th);
  (void)hipFree(coef);
  if (d_idx) (void)hipFree(d_idx);
  if (w) (void)hipFree(w);
  if (e != hipSuccess) {
    if (slab) (void)hipFree(slab);
    gwl_event_destroy(ev);
    return hip_fail(e, "relative-binning tables");
  }
  // the event now walks the edges
  (void)hipFree(ev->slab);
  ev->slab = slab;
  ev->ec = ec;
  ev->tab64 = tab64;
  ev->tab32 = tab32;
  ev->g32 = g32;
  ev->g64 = g64;
  ev->M_full = ev->M;
  ev->M = nedge;
  ev->M_loop = nedge;
  ev->rb_idx = idx;
  *out = ev;
  return GWL_OK;
}

// Calibration spline tables (host, float64): per bin the Catmull-Rom weights of the four nodes
// around it in ln f, with the linearly extrapolated ghost node beyond either end folded into
// the real end nodes, expressed over the interval's window of four real nodes; the interval
// starts; and per detector K1_j = sum_k K_k w_kj, K2_jl = sum_k K_k w_kj w_kl, K_k = 4 df
// f_k^-7/3 / S_k.
// Catmull-Rom weights of nodes j-1 .. j+2 on interval j as polynomials in t (coefficients of
// t^0 .. t^3), and the ghost nodes at both ends (-1 = 2 v0 - v1, n = 2 v_{n-1} - v_{n-2}) folded
// into the window of four nodes j0[j] .. j0[j] + 3: B[(j * 4 + i) * 4 + p].
static void cal_basis(int n, const int* j0, std::vector<double>& B) {
  const double C[4][4] = {{0.0, -0.5, 1.0, -0.5}, {1.0, 0.0, -2.5, 1.5}, {0.0, 0.5, 2.0, -1.5}, {0.0, 0.0, -0.5, 0.5}};
  B.assign((size_t)(n - 1) * 16, 0.0);
  for (int j = 0; j < n - 1; ++j) {
    double wn[MAXNODE + 2][4] = {};  // over nodes -1 .. n
    for (int i = 0; i < 4; ++i)
      for (int q = 0; q < 4; ++q) wn[j + i][q] += C[i][q];
    for (int q = 0; q < 4; ++q) {
      wn[1][q] += 2.0 * wn[0][q];
      wn[2][q] -= wn[0][q];
      wn[n][q] += 2.0 * wn[n + 1][q];
      wn[n - 1][q] -= wn[n + 1][q];
    }
    for (int i = 0; i < 4; ++i)
      for (int q = 0; q < 4; ++q) B[((size_t)j * 4 + i) * 4 + q] = wn[j0[j] + i + 1][q];
  }
}

static void cal_tables(const std::vector<double>& f, const std::vector<double>& psd, int nd, double df, int n,
                       std::vector<double>& w, std::vector<double>& tloc, int* j0, int64_t* kb,
                       std::vector<double>& kcal) {
  const int64_t M = (int64_t)f.size();
  const double x0 = log(f.front()), x1 = log(f.back());
  const double h = n > 1 ? (x1 - x0) / (n - 1) : 1.0;
  w.assign((size_t)M * 4, 0.0);
  tloc.assign((size_t)M, 0.0);
  std::vector<double> W((size_t)M * n, 0.0);  // weights over all nodes (for K1, K2)
  for (int j = 0; j < n - 1; ++j) j0[j] = std::min(std::max(j - 1, 0), n - 4);
  for (int64_t k = 0; k < M; ++k) {
    double s = (log(f[k]) - x0) / h;
    s = std::min(std::max(s, 0.0), (double)(n - 1));
    const int j = std::min(std::max((int)floor(s), 0), n - 2);
    const double t = s - j;
    tloc[(size_t)k] = t;
    double cw[4] = {0.5 * (-t + 2 * t * t - t * t * t), 0.5 * (2 - 5 * t * t + 3 * t * t * t),
                    0.5 * (t + 4 * t * t - 3 * t * t * t), 0.5 * (-t * t + t * t * t)};  // nodes j-1 .. j+2
    double wn[MAXNODE + 2] = {};  // over nodes -1 .. n
    for (int i = 0; i < 4; ++i) wn[j - 1 + i + 1] += cw[i];
    wn[1] += 2.0 * wn[0];          // ghost -1 = 2 v0 - v1
    wn[2] -= wn[0];
    wn[n] += 2.0 * wn[n + 1];      // ghost n = 2 v_{n-1} - v_{n-2}
    wn[n - 1] -= wn[n + 1];
    for (int i = 0; i < 4; ++i) w[(size_t)k * 4 + i] = wn[j0[j] + i + 1];
    for (int i = 0; i < n; ++i) W[(size_t)k * n + i] = wn[i + 1];
  }
  std::vector<int64_t> first;
  cal_intervals(f, n, first);
  for (int j = 0; j < n; ++j) kb[j] = first[(size_t)j];
  kcal.assign((size_t)nd * (n + n * n), 0.0);
  for (int d = 0; d < nd; ++d) {
    double* K1 = kcal.data() + (size_t)d * (n + n * n);
    double* K2 = K1 + n;
    for (int64_t k = 0; k < M; ++k) {
      const double Kk = 4.0 * df * pow(f[k], -7.0 / 3.0) / psd[(size_t)d * M + k];
      const double* Wk = W.data() + (size_t)k * n;
      for (int i = 0; i < n; ++i) {
        if (Wk[i] == 0.0) continue;
        K1[i] += Kk * Wk[i];
        for (int l = 0; l < n; ++l) K2[i * n + l] += Kk * Wk[i] * Wk[l];
      }
    }
  }
}

}  // extern "C"

namespace gwl {

// Attach calibration tables to an event whose bin loop walks rows at the frequencies `frow`
// (the grid itself, or relative-binning edges): per row the spline weights of its window and its
// position in its node interval, the interval starts in rows, the per-interval cubic basis; the
// spline moments K1, K2 of <h_cal|h_cal> always over every grid bin (fgrid, psd).
static gwl_status attach_cal(gwl_event ev, const std::vector<double>& frow, const std::vector<double>& fgrid,
                             const std::vector<double>& psd, int nnode) {
  const int ndet = ev->ndet;
  const int64_t M = (int64_t)frow.size();
  std::vector<double> w, tl, kc, kc_rows, basis, wfull, tfull;
  int j0full[MAXNODE];
  int64_t kbfull[MAXNODE];
  if (&frow == &fgrid) {
    cal_tables(fgrid, psd, ndet, ev->df, nnode, w, tl, ev->cal_j0, ev->cal_kb, kc);
  } else {
    // the rows' weights (their spline moments are not used: any positive PSD will do), then the
    // moments over the grid
    const std::vector<double> psd_rows((size_t)M * ndet, 1.0);
    cal_tables(frow, psd_rows, ndet, ev->df, nnode, w, tl, ev->cal_j0, ev->cal_kb, kc_rows);
    cal_tables(fgrid, psd, ndet, ev->df, nnode, wfull, tfull, j0full, kbfull, kc);
  }
  cal_basis(nnode, ev->cal_j0, basis);
  std::vector<RowCal32> w32((size_t)M);
  for (int64_t k = 0; k < M; ++k)
    for (int i = 0; i < 4; ++i) w32[(size_t)k].w[i] = (float)w[(size_t)k * 4 + i];
  // TAB_PAD zero rows past the last bin: the bin loops request rows ahead of their bin
  w32.resize((size_t)(M + TAB_PAD));
  for (int64_t k = M; k < M + TAB_PAD; ++k)
    for (int i = 0; i < 4; ++i) w32[(size_t)k].w[i] = 0.0f;
  w.resize((size_t)(M + TAB_PAD) * 4, 0.0);
  tl.resize((size_t)(M + TAB_PAD), 0.0);
  std::vector<float> t32(tl.begin(), tl.end());
  // the band-limited rows that follow: their interval's cubic at their own frequency, also a little
  // beyond the interval's ends
  const double x0 = log(frow.front()), hx = (log(frow.back()) - x0) / (nnode - 1);
  for (size_t r = 0; r < ev->band_f.size(); ++r) {
    const int j = ev->band_seg[r];
    const double t = (log(ev->band_f[r]) - x0) / hx - j;
    tl.push_back(t);
    for (int i = 0; i < 4; ++i) {
      const double* Bi = &basis[((size_t)j * 4 + i) * 4];
      w.push_back(fma(fma(fma(Bi[3], t, Bi[2]), t, Bi[1]), t, Bi[0]));
    }
  }
  if (!ev->band_f.empty()) {
    tl.resize(tl.size() + TAB_PAD, 0.0);
    w.resize(w.size() + TAB_PAD * 4, 0.0);
  }
  std::vector<double>().swap(ev->band_f);
  std::vector<int>().swap(ev->band_seg);
  ev->cal_slope = cal_slope(cal_reach(hx)) / (2.0 * M_PI * hx);
  Slab keep;
  const size_t o32 = keep.take(sizeof(RowCal32) * (M + TAB_PAD)), o64 = keep.take(sizeof(double) * w.size());
  const size_t ot32 = keep.take(sizeof(float) * (M + TAB_PAD)), ot64 = keep.take(sizeof(double) * tl.size());
  const size_t ob = keep.take(sizeof(double) * basis.size()), ok = keep.take(sizeof(double) * kc.size());
  char* slab = nullptr;
  hipError_t e = hipMalloc((void**)&slab, keep.bytes);
  if (e == hipSuccess) {
    ev->cal_slab = slab;
    ev->cal32 = (RowCal32*)(slab + o32);
    ev->cal64 = (RowCal64*)(slab + o64);
    ev->calt32 = (float*)(slab + ot32);
    ev->calt64 = (double*)(slab + ot64);
    ev->calB = (double*)(slab + ob);
    ev->kcal = (double*)(slab + ok);
  }
  if (e == hipSuccess) e = hipMemcpy(ev->cal32, w32.data(), sizeof(RowCal32) * (M + TAB_PAD), hipMemcpyHostToDevice);
  if (e == hipSuccess) e = hipMemcpy(ev->cal64, w.data(), sizeof(double) * w.size(), hipMemcpyHostToDevice);
  if (e == hipSuccess) e = hipMemcpy(ev->calt32, t32.data(), sizeof(float) * (M + TAB_PAD), hipMemcpyHostToDevice);
  if (e == hipSuccess) e = hipMemcpy(ev->calt64, tl.data(), sizeof(double) * tl.size(), hipMemcpyHostToDevice);
  if (e == hipSuccess) e = hipMemcpy(ev->calB, basis.data(), sizeof(double) * basis.size(), hipMemcpyHostToDevice);
  if (e == hipSuccess) e = hipMemcpy(ev->kcal, kc.data(), sizeof(double) * kc.size(), hipMemcpyHostToDevice);
  if (e != hipSuccess) return hip_fail(e, "calibration tables");
  ev->ncal = nnode;
  return GWL_OK;
}

static gwl_status read_grid(const double* fgrid, const double* psd, int ndet, int64_t M, hipStream_t s,
                            std::vector<double>& fh, std::vector<double>& ph) {
  fh.resize((size_t)M);
  ph.resize((size_t)M * ndet);
  hipError_t e = hipMemcpyAsync(fh.data(), fgrid, sizeof(double) * M, hipMemcpyDeviceToHost, s);
  if (e == hipSuccess) e = hipMemcpyAsync(ph.data(), psd, sizeof(double) * M * ndet, hipMemcpyDeviceToHost, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  if (e != hipSuccess) return hip_fail(e, "grid read-back");
  return GWL_OK;
}

}  // namespace gwl

extern "C" {

gwl_status gwl_event_create_cal(const double* data, const double* psd, const gwl_detector* dets, int ndet,
                                const double* fgrid, int64_t M, double df, double gmst, int nnode, unsigned flags,
                                void* stream, gwl_event* out) {
  clear_error();
  if (!out) return fail(GWL_E_INVALID, "out is null");
  *out = nullptr;
  if (nnode < 4 || nnode > MAXNODE) return fail(GWL_E_SHAPE, "nnode=%d outside [4, %d]", nnode, MAXNODE);
  if (flags & GWL_F_ISCO_CUTOFF)
    return fail(GWL_E_UNSUPPORTED, "the ISCO cut-off is not available with the calibration model");
  gwl_event ev = nullptr;
  gwl_status st = event_create(data, psd, dets, ndet, fgrid, M, df, gmst, flags, stream, true, nnode, &ev);
  if (st != GWL_OK) return st;
  std::vector<double> fh, ph;
  st = read_grid(fgrid, psd, ndet, M, (hipStream_t)stream, fh, ph);
  if (st == GWL_OK) st = attach_cal(ev, fh, fh, ph, nnode);
  if (st != GWL_OK) {
    gwl_event_destroy(ev);
    return st;
  }
  *out = ev;
  return GWL_OK;
}

gwl_status gwl_event_create_rb_cal(const double* data, const double* psd, const gwl_detector* dets, int ndet,
                                   const double* fgrid, int64_t M, double df, double gmst, const double* theta_fid,
                                   double eps, int nnode, unsigned flags, void* stream, gwl_event* out) {
  clear_error();
  if (!out) return fail(GWL_E_INVALID, "out is null");
  *out = nullptr;
  if (nnode < 4 || nnode > MAXNODE) return fail(GWL_E_SHAPE, "nnode=%d outside [4, %d]", nnode, MAXNODE);
  gwl_event ev = nullptr;
  gwl_status st = gwl_event_create_rb(data, psd, dets, ndet, fgrid, M, df, gmst, theta_fid, eps, flags, stream, &ev);
  if (st != GWL_OK) return st;
  std::vector<double> fh, ph;
  st = read_grid(fgrid, psd, ndet, M, (hipStream_t)stream, fh, ph);
  if (st == GWL_OK) {
    std::vector<double> fe(ev->rb_idx.size());
    for (size_t i = 0; i < fe.size(); ++i) fe[i] = fh[(size_t)ev->rb_idx[i]];
    st = attach_cal(ev, fe, fh, ph, nnode);
  }
  if (st != GWL_OK) {
    gwl_event_destroy(ev);
    return st;
  }
  *out = ev;
  return GWL_OK;
}

gwl_status gwl_event_destroy(gwl_event ev) {
  if (!ev) return GWL_OK;
  for (gwl_workspace& w : ev->ws) {
    if (w.ptr) (void)hipFree(w.ptr);
    if (w.cnt) (void)hipFree(w.cnt);
  }
  ev->ws.clear();
  if (ev->cal_slab) (void)hipFree(ev->cal_slab);
  if (ev->slab) (void)hipFree(ev->slab);
  if (ev->fgrid) (void)hipFree(ev->fgrid);
  if (ev->kcum) (void)hipFree(ev->kcum);
  delete ev;
  return GWL_OK;
}

gwl_status gwl_event_rb_info(gwl_event ev, int64_t* nedge, int64_t* nbins) {
  clear_error();
  if (!ev) return fail(GWL_E_INVALID, "event is null");
  if (nedge) *nedge = ev->M_full ? ev->M : 0;
  if (nbins) *nbins = ev->M_full ? ev->M_full : ev->M;
  return GWL_OK;
}

gwl_status gwl_event_info(gwl_event ev, int* ndet, int64_t* M, double* df) {
  clear_error();
  if (!ev) return fail(GWL_E_INVALID, "event is null");
  if (ndet) *ndet = ev->ndet;
  if (M) *M = ev->M;
  if (df) *df = ev->df;
  return GWL_OK;
}

}  // extern "C"

namespace gwl {

// Launch shape of a calibrated call: every point group's rows in nchunk equal shares, one wavefront
// each.
static CalShape cal_shape(const gwl_event_s* ev, int64_t B, bool grad) {
  CalShape sh;
  memset(&sh, 0, sizeof sh);
  const int n = ev->ncal;
  sh.nnode = n;
  sh.npg = (int)((B + WAVE - 1) / WAVE);
  // Workgroups of four chunks resident together, by the loops' registers (four wavefronts per SIMD for values,
  // two for three detectors' gradients; a part-filled second round costs a whole one): as many of them as fit, or one a
  // group more where that leaves a quarter of them empty, and 48 rows a chunk at least (the epilogue walks the
  // chunks in turn). Three detectors, 8 s, 10 nodes, with as many as make 4,096 wavefronts (gradients 2,048) of
  // 24 rows and now: values of 1,000 points 62 and 55 us, 9,000 123 and 102, 20,000 198 and 172; gradients
  // of 1,000 135 and 95, 5,000 153 and 129. (At 12, 24, 40, 60 and 90 rows gradients of 1,000 points take
  // 172, 135, 101, 93 and 94, values of 3,000 78, 78, 72, 69 and 79.)
  const int64_t fit = grad ? (ev->ndet == 1 ? 1024 : (ev->ndet == 2 ? 768 : 512)) : 1024;
  int64_t nbc = std::max<int64_t>(1, fit / sh.npg);
  if (4 * nbc * sh.npg < 3 * fit) ++nbc;
  sh.nchunk = (int)std::max<int64_t>(1, std::min<int64_t>({WAVES_PER_BLOCK * nbc, ev->M_loop / 48, 128}));
  sh.nbc = (sh.nchunk + WAVES_PER_BLOCK - 1) / WAVES_PER_BLOCK;
  sh.items = sh.npg * sh.nbc;
  sh.gper = (sh.items + NXCD - 1) / NXCD;
  for (int j = 0; j < n - 1; ++j) sh.j0[j] = ev->cal_j0[j];
  for (int j = 0; j < n; ++j) sh.k0[j] = (int)ev->cal_kb[j];
  return sh;
}

// Launch shape of a live-length call.
LoopShape live_shape(const gwl_event_s* ev, int64_t B, bool mixed) {
  // On band-limited rows: eight wavefronts a workgroup, of which two are resident on a CU, and as many
  // workgroups a point group as are resident with all of the batch live (16 rows a wavefront at
  // least). 8,192 points of three detectors and 8 s at 10, 40, 60 and 100 % live: 34, 35, 45 and 45 us;
  // twice as many workgroups 29, 35, 47 and 57, half as many 46 to 47.
  LoopShape sh = make_shape(B, ev->M, 8, 1, 1, 1);
  const int64_t fill = std::max<int64_t>(1, 2 * 256 / sh.npg), most = std::max<int64_t>(1, ev->M_loop / (16 * 8));
  sh = make_shape(B, ev->M, 8, (int)std::min(fill, most), 1, 1);
  if (ev->nlev[mixed] > 0 && sh.chunk > kBandMinChunk) {
    sh.levels = 1;
    return sh;
  }
  // On the bins: the shape for B, with at least enough workgroups per point group that a quarter of the
  // point groups still give every CU two workgroups (chunks of at least 16 bins): a partly live batch
  // then still fills the chip. The G workgroup sums go to the separate epilogue kernel (the
  // set-up in either kernel): at these workgroup counts the last-arriver's device-scope fences
  // cost more than the second launch (on c1 shapes with 8192 points, 240 against 196 us)
  sh = choose_shape(ev, B, mixed, false);
  const int64_t want = (4 * 2 * 256 + sh.npg - 1) / sh.npg;
  const int64_t gcap = std::max<int64_t>(1, ev->M / (32 * (int64_t)sh.W));
  const int G = (int)std::min<int64_t>(std::max<int64_t>(sh.G, want), std::max<int64_t>(gcap, sh.G));
  sh = make_shape(B, ev->M, sh.W, G, sh.setup, 1);
  return sh;
}

// set-up rows, calibration rows, sums per chunk, window moments per piece, a plan per point group
static size_t cal_bytes(const gwl_event_s* ev, const CalShape& sh, bool grad, bool order) {
  const size_t Bp = (size_t)sh.npg * WAVE, nd = ev->ndet, n = ev->ncal;
  return sizeof(double) * Bp * (NCOEF + 2 * n * nd + sh.nchunk * (size_t)nz_of((int)nd, grad) +
                                (sh.nchunk + n - 2) * (size_t)nz_win((int)nd, grad)) +
         sizeof(int) * PLAN_INTS * (size_t)sh.npg + (order ? sizeof(int) * Bp : 0);
}

// The plans in that workspace.
static int* cal_plan(const gwl_event_s* ev, const CalShape& sh, bool grad, void* ws) {
  return (int*)((char*)ws + cal_bytes(ev, sh, grad, false)) - (size_t)PLAN_INTS * sh.npg;
}

}  // namespace gwl

extern "C" {

// Calibrated evaluation, in the event's workspace for s, or (a multi-event plan) in ws_given of
// ws_bytes bytes, owned by the caller.
static gwl_status run_logl_cal(gwl_event ev, const double* theta, int64_t B, bool mixed, bool grad, double* logl,
                               double* gradout, hipStream_t s, void* ws_given = nullptr, size_t ws_bytes = 0) {
  const int nd = ev->ndet, n = ev->ncal;
  const CalShape sh = cal_shape(ev, B, grad);
  const int64_t Bp = (int64_t)sh.npg * WAVE;
  const int ncal = 2 * n * nd;
  bool order = in_order(ev, B, grad, INT_MAX);
  size_t bytes = cal_bytes(ev, sh, grad, order);
  void* ws = ws_given;
  if (ws_given) {
    if (ws_bytes < bytes) return fail(GWL_E_INTERNAL, "calibrated loop: workspace of %zu bytes, %zu needed", ws_bytes, bytes);
  } else {
    gwl_status st = event_workspace(ev, s, bytes, 0, &ws);
    if (st != GWL_OK && order) {                       // no room for the order: the caller's own
      clear_error();
      order = false;
      bytes = cal_bytes(ev, sh, grad, order);
      st = event_workspace(ev, s, bytes, 0, &ws);
    }
    if (st != GWL_OK) return st;
  }
  double* coef = (double*)ws;
  double* calc = coef + (size_t)NCOEF * Bp;
  double* part = calc + (size_t)ncal * Bp;
  int* plan = cal_plan(ev, sh, grad, ws);
  const CalTables t = {ev->tab64, ev->tab32, ev->g64, ev->g32, ev->cal64, ev->cal32, ev->calt64, ev->calt32, ev->calB,
                       ev->kcal, ev->bands, ev->cal_slope};
  int* perm = order ? plan + (size_t)PLAN_INTS * sh.npg : nullptr;
  hipError_t e = perm ? launch_order(theta, NPARAM + ncal, B, perm, s) : hipSuccess;
  if (e == hipSuccess)
    e = launch_cal(nd, mixed, grad, ev->geom, ev->ec, t, theta, NPARAM + ncal, B, Bp, ev->M, sh, coef, calc, part, plan,
                   perm, logl, gradout, s);
  if (e != hipSuccess) return hip_fail(e, "launch");
  return GWL_OK;
}

static gwl_status logl_common(gwl_event ev, const double* theta, int64_t B, gwl_precision prec, double* logl,
                              double* grad, bool with_grad, void* stream) {
  clear_error();
  if (!ev) return fail(GWL_E_INVALID, "event is null");
  if (B < 0 || B > kMaxBatch) return fail(GWL_E_SHAPE, "B=%lld outside [0, %lld]", (long long)B, (long long)kMaxBatch);
  if (prec != GWL_FP64 && prec != GWL_MIXED) return fail(GWL_E_INVALID, "unknown precision %d", (int)prec);
  if (B == 0) return GWL_OK;
  if (!theta || !logl || (with_grad && !grad)) return fail(GWL_E_INVALID, "theta, logl%s must be device pointers",
                                                           with_grad ? " and grad" : "");
  gwl_status st = check_device(ev->device);
  if (st != GWL_OK) return st;
  const bool mixed = use_mixed(ev, prec);
  if (ev->ncal > 0) return run_logl_cal(ev, theta, B, mixed, with_grad, logl, grad, (hipStream_t)stream);
  const LoopShape sh = choose_shape(ev, B, mixed, with_grad);
  return run_logl(ev, theta, B, mixed, with_grad, sh, logl, grad, (hipStream_t)stream);
}

gwl_status gwl_logl_batch(gwl_event ev, const double* theta, int64_t B, gwl_precision prec, double* logl,
                          void* stream) {
  return logl_common(ev, theta, B, prec, logl, nullptr, false, stream);
}

gwl_status gwl_logl_batch_live(gwl_event ev, const double* theta, int64_t B, const int64_t* live, gwl_precision prec,
                               double* logl, void* stream) {
  clear_error();
  if (!ev) return fail(GWL_E_INVALID, "event is null");
  if (B < 0 || B > kMaxBatch) return fail(GWL_E_SHAPE, "B=%lld outside [0, %lld]", (long long)B, (long long)kMaxBatch);
  if (prec != GWL_FP64 && prec != GWL_MIXED) return fail(GWL_E_INVALID, "unknown precision %d", (int)prec);
  if (!live) return fail(GWL_E_INVALID, "live must be a device pointer");
  if (B == 0) return GWL_OK;
  if (!theta || !logl) return fail(GWL_E_INVALID, "theta and logl must be device pointers");
  if (ev->ncal > 0) return fail(GWL_E_UNSUPPORTED, "gwl_logl_batch_live does not take calibrated events");
  gwl_status st = check_device(ev->device);
  if (st != GWL_OK) return st;
  const bool mixed = use_mixed(ev, prec);
  const LoopShape sh = live_shape(ev, B, mixed);
  return run_logl(ev, theta, B, mixed, false, sh, logl, nullptr, (hipStream_t)stream, live);
}

gwl_status gwl_logl_grad(gwl_event ev, const double* theta, int64_t B, gwl_precision prec, double* logl, double* grad,
                         void* stream) {
  return logl_common(ev, theta, B, prec, logl, grad, true, stream);
}

gwl_status gwl_event_reserve(gwl_event ev, int64_t B, gwl_precision prec, int with_grad, void* stream) {
  clear_error();
  if (!ev) return fail(GWL_E_INVALID, "event is null");
  if (B < 0 || B > kMaxBatch) return fail(GWL_E_SHAPE, "B=%lld outside [0, %lld]", (long long)B, (long long)kMaxBatch);
  if (prec != GWL_FP64 && prec != GWL_MIXED) return fail(GWL_E_INVALID, "unknown precision %d", (int)prec);
  if (B == 0) return GWL_OK;
  gwl_status st = check_device(ev->device);
  if (st != GWL_OK) return st;
  void* ws = nullptr;
  const bool mixed = use_mixed(ev, prec), grad = with_grad != 0;
  size_t bytes = call_workspace_bytes(ev, B, mixed, grad), ncnt = 0;
  if (ev->ncal == 0) ncnt = workspace_counters(choose_shape(ev, B, mixed, grad), grad);
  if (ev->ncal == 0 && !grad) {                        // a live-length call of this size, whose shape is its own
    const LoopShape sh = live_shape(ev, B, mixed);
    bytes = std::max(bytes, workspace_bytes((int64_t)sh.npg * WAVE, sh, ev->ndet, false));
    ncnt = std::max(ncnt, workspace_counters(sh, false));
  }
  return event_workspace(ev, (hipStream_t)stream, bytes, ncnt, &ws);
}

gwl_status gwl_launch_shape(gwl_event ev, int64_t B, gwl_precision prec, int with_grad, int* nchunk,
                            int* chunk_bins) {
  clear_error();
  if (!ev) return fail(GWL_E_INVALID, "event is null");
  if (B < 1 || B > kMaxBatch) return fail(GWL_E_SHAPE, "B=%lld outside [1, %lld]", (long long)B, (long long)kMaxBatch);
  if (prec != GWL_FP64 && prec != GWL_MIXED) return fail(GWL_E_INVALID, "unknown precision %d", (int)prec);
  const LoopShape sh = choose_shape(ev, B, use_mixed(ev, prec), with_grad != 0);
  if (nchunk) *nchunk = sh.nchunk;
  if (chunk_bins) *chunk_bins = sh.chunk;
  return GWL_OK;
}

gwl_status gwl_launch_layout(gwl_event ev, int64_t B, gwl_precision prec, int with_grad, int* waves, int* groups,
                             int* setup) {
  clear_error();
  if (!ev) return fail(GWL_E_INVALID, "event is null");
  if (B < 1 || B > kMaxBatch) return fail(GWL_E_SHAPE, "B=%lld outside [1, %lld]", (long long)B, (long long)kMaxBatch);
  if (prec != GWL_FP64 && prec != GWL_MIXED) return fail(GWL_E_INVALID, "unknown precision %d", (int)prec);
  const LoopShape sh = choose_shape(ev, B, use_mixed(ev, prec), with_grad != 0);
  if (waves) *waves = sh.W;
  if (groups) *groups = sh.G;
  if (setup) *setup = sh.setup;
  return GWL_OK;
}

gwl_status gwl_call_rows(gwl_event ev, const double* theta, int64_t B, gwl_precision prec, int with_grad,
                         int64_t* float64_rows, int64_t* mixed_bins, void* stream) {
  clear_error();
  if (!ev) return fail(GWL_E_INVALID, "event is null");
  if (B < 0 || B > kMaxBatch) return fail(GWL_E_SHAPE, "B=%lld outside [0, %lld]", (long long)B, (long long)kMaxBatch);
  if (prec != GWL_FP64 && prec != GWL_MIXED) return fail(GWL_E_INVALID, "unknown precision %d", (int)prec);
  if (B > 0 && !theta) return fail(GWL_E_INVALID, "theta must be a device pointer");
  gwl_status st = check_device(ev->device);
  if (st != GWL_OK) return st;
  const bool mixed = use_mixed(ev, prec), grad = with_grad != 0, cal = ev->ncal > 0;
  hipStream_t s = (hipStream_t)stream;
  int64_t n[2] = {0, 0};                               // float64 rows, mixed bins
  const LoopShape sh = choose_shape(ev, std::max<int64_t>(B, 1), mixed, grad);
  if (B > 0 && ev->bands && (cal || sh.chunk > kBandMinChunk)) {
    const CalShape cs = cal ? cal_shape(ev, B, grad) : CalShape{};
    const int64_t npg = (B + WAVE - 1) / WAVE, Bp = npg * WAVE, P = NPARAM + 2 * ev->ncal * ev->ndet;
    const bool order = cal ? in_order(ev, B, grad, INT_MAX) : sh.order != 0;
    Slab slab;
    const size_t ows = slab.take(cal ? cal_bytes(ev, cs, grad, order) : sizeof(double) * NCOEF * (size_t)Bp);
    const size_t oplan = slab.take(sizeof(int) * PLAN_INTS * (size_t)npg), operm = slab.take(sizeof(int) * (size_t)Bp);
    const size_t oout = slab.take(cal ? sizeof(double) * (size_t)(B * (grad ? P + 1 : 1)) : 0);
    char* p = nullptr;
    hipError_t e = hipMalloc((void**)&p, slab.bytes);
    int* plan = (int*)(p + oplan);
    if (e == hipSuccess && cal) {                      // the whole call: its plans stay in its workspace
      st = run_logl_cal(ev, theta, B, mixed, grad, (double*)(p + oout), (double*)(p + oout) + B, s, p + ows,
                        cal_bytes(ev, cs, grad, order));
      plan = cal_plan(ev, cs, grad, p + ows);
    } else if (e == hipSuccess) {
      int* perm = order ? (int*)(p + operm) : nullptr;
      if (perm) e = launch_order(theta, NPARAM, B, perm, s);
      if (e == hipSuccess)
        e = launch_setup(ev->ndet, ev->geom, ev->ec, theta, B, Bp, (double*)(p + ows), s, ev->bands,
                         float64_most(mixed, grad, false, ev->M), 1, plan, perm);
    }
    std::vector<int> h((size_t)npg * PLAN_INTS);
    if (e == hipSuccess && st == GWL_OK)
      e = hipMemcpyAsync(h.data(), plan, sizeof(int) * h.size(), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (p) (void)hipFree(p);
    if (e != hipSuccess) return hip_fail(e, "rows of a call");
    if (st != GWL_OK) return st;
    for (int64_t g = 0; g < npg; ++g) {
      const int* pl = &h[(size_t)g * PLAN_INTS];
      n[pl[2] ? 0 : 1] += std::min<int64_t>(WAVE, B - g * WAVE) * (pl[2] ? pl[0] : ev->M);
    }
  } else {
    n[mixed ? 1 : 0] = B * ev->M;
  }
  if (float64_rows) *float64_rows = n[0];
  if (mixed_bins) *mixed_bins = n[1];
  return GWL_OK;
}

gwl_status gwl_waveform(const double* theta, int64_t B, const gwl_detector* dets, int ndet, const double* fgrid,
                        int64_t M, double gmst, double* out, void* stream) {
  clear_error();
  EventGeom g;
  gwl_status st = make_geom(dets, ndet, gmst, g);
  if (st != GWL_OK) return st;
  if (B < 0 || B > 65535) return fail(GWL_E_SHAPE, "B=%lld outside [0, 65535]", (long long)B);
  if (M < 1 || M > (int64_t)1 << 30) return fail(GWL_E_SHAPE, "M=%lld outside [1, 2^30]", (long long)M);
  if (B == 0) return GWL_OK;
  if (!theta || !fgrid || !out) return fail(GWL_E_INVALID, "theta, fgrid and out must be device pointers");
  hipStream_t s = (hipStream_t)stream;
  const int64_t Bp = (B + WAVE - 1) / WAVE * WAVE;
  double* coef = nullptr;
  hipError_t e = hipMallocAsync((void**)&coef, sizeof(double) * NCOEF * (size_t)Bp, s);
  if (e != hipSuccess) return hip_fail(e, "workspace");
  e = launch_setup(ndet, g, nullptr, theta, B, Bp, coef, s);
  if (e == hipSuccess) e = launch_waveform(ndet, g, coef, B, Bp, fgrid, M, out, s);
  hipError_t e2 = hipFreeAsync(coef, s);
  if (e != hipSuccess) return hip_fail(e, "waveform launch");
  if (e2 != hipSuccess) return hip_fail(e2, "workspace release");
  return GWL_OK;
}

}  // extern "C"

namespace gwl {

gwl_status run_calibrated(gwl_event ev, const double* theta, int64_t B, bool mixed, bool grad, double* logl,
                          double* gradout, hipStream_t s, void* ws, size_t ws_bytes) {
  return run_logl_cal(ev, theta, B, mixed, grad, logl, gradout, s, ws, ws_bytes);
}

// The set-up rows [NCOEF][Bp] come first unless the evaluation kernel makes them itself and
// nothing after it reads them (with the separate value epilogue it leaves that kernel's rows there)
static bool coef_in_workspace(const LoopShape& sh, bool grad) { return !sh.setup || (!grad && sh.G > 1 && sh.sepepi); }

size_t workspace_bytes(int64_t Bp, const LoopShape& sh, int nd, bool grad) {
  const size_t coef = coef_in_workspace(sh, grad) ? (size_t)NCOEF * Bp : 0;
  const size_t part = (grad || sh.G > 1) ? (size_t)sh.G * nz_of(nd, grad) * Bp : 0;
  const size_t plan = sh.setup ? 0 : sizeof(int) * PLAN_INTS * (size_t)(Bp / WAVE);
  return sizeof(double) * (coef + part) + plan + (sh.order ? sizeof(int) * (size_t)Bp : 0);
}

size_t workspace_counters(const LoopShape& sh, bool grad) {
  return (!grad && sh.G > 1 && !sh.sepepi) ? (size_t)sh.npg : 0;
}

// Set-up, bin loop and epilogue on `s`, in the event's workspace for `s`.
gwl_status run_logl(gwl_event ev, const double* theta, int64_t B, bool mixed, bool grad, const LoopShape& shape,
                    double* logl, double* gradout, hipStream_t s, const int64_t* live) {
  LoopShape sh = shape;
  const int64_t Bp = (int64_t)sh.npg * WAVE;
  void* ws = nullptr;
  unsigned int* cnt = nullptr;
  gwl_status st = event_workspace(ev, s, workspace_bytes(Bp, sh, ev->ndet, grad), workspace_counters(sh, grad), &ws,
                                  &cnt);
  if (st != GWL_OK && sh.order) {                      // no room for the order: the caller's own
    clear_error();
    sh.order = 0;
    st = event_workspace(ev, s, workspace_bytes(Bp, sh, ev->ndet, grad), workspace_counters(sh, grad), &ws, &cnt);
  }
  if (st != GWL_OK) return st;
  hipError_t e = enqueue_logl(ev, theta, B, mixed, grad, sh, (double*)ws, cnt, logl, gradout, s, live);
  if (e != hipSuccess) return hip_fail(e, "launch");
  return GWL_OK;
}

gwl_status event_workspace(gwl_event ev, hipStream_t s, size_t bytes, size_t ncnt, void** out, unsigned int** cnt) {
  *out = nullptr;
  if (cnt) *cnt = nullptr;
  std::lock_guard<std::mutex> lk(ev->ws_mu);
  gwl_workspace* w = nullptr;
  for (gwl_workspace& x : ev->ws)
    if (x.stream == s) w = &x;
  if (w && w->bytes >= bytes && w->ncnt >= ncnt) {
    *out = w->ptr;
    if (cnt) *cnt = w->cnt;
    return GWL_OK;
  }
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  hipError_t e = hipStreamIsCapturing(s, &cs);
  if (e != hipSuccess) return hip_fail(e, "stream capture status");
  if (cs != hipStreamCaptureStatusNone)
    return fail(GWL_E_INVALID, "the call needs %zu bytes of workspace on a stream that is capturing a graph and has %zu: "
                               "reserve it first (gwl_event_reserve, or one call of this size on that stream outside "
                               "capture)", bytes, w ? w->bytes : (size_t)0);
  if (!w) {
    ev->ws.push_back(gwl_workspace{});
    w = &ev->ws.back();
    w->stream = s;
  }
  const size_t grain = (size_t)2 << 20;
  const size_t nb = std::max(w->bytes, (bytes + grain - 1) / grain * grain);
  const size_t nc = std::max(w->ncnt, (ncnt + 1023) / 1024 * 1024);
  void* p = w->ptr;
  unsigned int* c = w->cnt;
  if (nb > w->bytes) {
    e = hipMalloc(&p, nb);
    if (e != hipSuccess) return hip_fail(e, "workspace");
  }
  if (nc > w->ncnt) {
    e = hipMalloc((void**)&c, nc * sizeof(unsigned int));
    // the kernels leave their counters at zero; a new array starts there
    if (e == hipSuccess) e = hipMemsetAsync(c, 0, nc * sizeof(unsigned int), s);
  }
  // buffers being replaced may still be in use by work queued on s
  const bool replace_ptr = p != w->ptr && w->ptr, replace_cnt = c != w->cnt && w->cnt;
  if (e == hipSuccess && (replace_ptr || replace_cnt)) e = hipStreamSynchronize(s);
  if (e != hipSuccess) {
    if (p != w->ptr) (void)hipFree(p);
    if (c != w->cnt && c) (void)hipFree(c);
    return hip_fail(e, "workspace");
  }
  if (replace_ptr) (void)hipFree(w->ptr);
  if (replace_cnt) (void)hipFree(w->cnt);
  w->ptr = p;
  w->bytes = nb;
  w->cnt = c;
  w->ncnt = nc;
  *out = p;
  if (cnt) *cnt = c;
  return GWL_OK;
}

size_t call_workspace_bytes(const gwl_event_s* ev, int64_t B, bool mixed, bool grad) {
  const int64_t Bp = (B + WAVE - 1) / WAVE * WAVE;
  if (ev->ncal > 0) return cal_bytes(ev, cal_shape(ev, B, grad), grad, in_order(ev, B, grad, INT_MAX));
  return workspace_bytes(Bp, choose_shape(ev, B, mixed, grad), ev->ndet, grad);
}

// ---- bin-loop timing (gwl_profile_*) ----
static std::mutex g_prof_mu;
static bool g_prof_on = false;
static std::vector<std::pair<hipEvent_t, hipEvent_t>> g_prof_events;

static bool prof_begin(hipStream_t s, hipEvent_t& a, hipEvent_t& b) {
  {
    std::lock_guard<std::mutex> lk(g_prof_mu);
    if (!g_prof_on) return false;
  }
  if (hipEventCreate(&a) != hipSuccess) return false;
  if (hipEventCreate(&b) != hipSuccess) {
    (void)hipEventDestroy(a);
    return false;
  }
  (void)hipEventRecord(a, s);
  return true;
}

static void prof_end(hipStream_t s, hipEvent_t a, hipEvent_t b) {
  (void)hipEventRecord(b, s);
  std::lock_guard<std::mutex> lk(g_prof_mu);
  g_prof_events.emplace_back(a, b);
}

hipError_t enqueue_logl(gwl_event ev, const double* theta, int64_t B, bool mixed, bool grad, const LoopShape& sh,
                        double* ws, unsigned int* cnt, double* logl, double* gradout, hipStream_t s,
                        const int64_t* live) {
  const int64_t Bp = (int64_t)sh.npg * WAVE;
  const bool with_coef = coef_in_workspace(sh, grad);
  double* coef = with_coef ? ws : nullptr;
  double* part = (grad || sh.G > 1) ? ws + (with_coef ? (size_t)NCOEF * Bp : 0) : nullptr;
  const size_t npart = (grad || sh.G > 1) ? (size_t)sh.G * nz_of(ev->ndet, grad) * Bp : 0;
  int* plan = sh.setup ? nullptr : (int*)(ws + (with_coef ? (size_t)NCOEF * Bp : 0) + npart);
  const BandHead* bands = (live ? sh.levels != 0 : sh.chunk > kBandMinChunk) ? ev->bands : nullptr;
  int* perm = sh.order && bands && !live
                  ? (int*)(ws + (with_coef ? (size_t)NCOEF * Bp : 0) + npart) + (sh.setup ? 0 : (size_t)PLAN_INTS * sh.npg)
                  : nullptr;
  hipError_t e = perm ? launch_order(theta, NPARAM, B, perm, s) : hipSuccess;
  if (e == hipSuccess && !sh.setup)
    e = launch_setup(ev->ndet, ev->geom, ev->ec, theta, B, Bp, coef, s, bands,
                     float64_most(mixed, grad, false, ev->M), sh.nchunk, plan, perm);
  hipEvent_t pa = nullptr, pb = nullptr;
  const bool prof = e == hipSuccess && prof_begin(s, pa, pb);
  const EvalArgs x = {ev->tab64, ev->tab32, ev->g64, theta, &ev->geom, ev->ec, bands, plan, coef, B, Bp, ev->M,
                      part, cnt, logl, ev->fgrid, ev->kcum, live, perm};
  if (e == hipSuccess) e = launch_eval(ev->ndet, mixed, grad, ev->ech.uniform != 0, x, sh, s);
  // the value's reduction over the G workgroups in its own kernel (timed with the evaluation)
  if (e == hipSuccess && !grad && sh.G > 1 && sh.sepepi)
    e = launch_value_epilogue(ev->ndet, ev->ec, theta, coef, B, Bp, sh.G, part, logl, ev->fgrid, ev->kcum, ev->M, live,
                              perm, s);
  if (prof) prof_end(s, pa, pb);
  if (e == hipSuccess && grad)
    e = launch_epilogue(ev->ndet, true, ev->geom, ev->ec, theta, coef, B, Bp, sh.G, part, logl, gradout, s, ev->fgrid,
                        ev->kcum, ev->M, perm);
  return e;
}

}  // namespace gwl

extern "C" {

gwl_status gwl_profile_enable(int on) {
  clear_error();
  std::lock_guard<std::mutex> lk(gwl::g_prof_mu);
  gwl::g_prof_on = on != 0;
  return GWL_OK;
}

gwl_status gwl_profile_read(int64_t* launches, double* total_ms) {
  clear_error();
  std::vector<std::pair<hipEvent_t, hipEvent_t>> ev;
  {
    std::lock_guard<std::mutex> lk(gwl::g_prof_mu);
    ev.swap(gwl::g_prof_events);
  }
  double tot = 0.0;
  hipError_t err = hipSuccess;
  for (auto& p : ev) {
    hipError_t e = hipEventSynchronize(p.second);
    float ms = 0.0f;
    if (e == hipSuccess) e = hipEventElapsedTime(&ms, p.first, p.second);
    if (e == hipSuccess) tot += ms;
    else if (err == hipSuccess) err = e;
    (void)hipEventDestroy(p.first);
    (void)hipEventDestroy(p.second);
  }
  if (launches) *launches = (int64_t)ev.size();
  if (total_ms) *total_ms = tot;
  if (err != hipSuccess) return hip_fail(err, "profile read");
  return GWL_OK;
}

}  // extern "C"
