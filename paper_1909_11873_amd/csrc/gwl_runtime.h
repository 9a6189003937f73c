// Internal host-side declarations shared by the runtime's translation units.
#pragma once

#include <hip/hip_runtime.h>

#include <mutex>
#include <vector>

#include "../../include/gwlike.h"
#include "gwl_bands.h"
#include "gwl_common.h"
#include "gwl_launch.h"

// Device workspace of an event on one stream: grown (never shrunk) outside graph capture, reused
// by every later call on that stream; calls on one stream are ordered, so they can share it.
struct gwl_workspace {
  hipStream_t stream = nullptr;
  void* ptr = nullptr;
  size_t bytes = 0;
  unsigned int* cnt = nullptr;       // completion counters of the evaluation kernel: zero between calls
  size_t ncnt = 0;
};

struct gwl_event_s {
  std::mutex ws_mu;                  // guards ws
  std::vector<gwl_workspace> ws;     // one per stream that has called on this event
  int device = 0;
  int ndet = 0;
  int64_t M = 0;                     // rows the bin loop walks (bins, or edges for relative binning)
  int64_t M_full = 0;                // bins of the grid (relative binning), else 0
  std::vector<int64_t> rb_idx;       // the relative-binning edges' bins
  // calibration model (ncal nodes per detector, 0 = none)
  int ncal = 0;
  gwl::RowCal32* cal32 = nullptr;    // [M] window weights
  gwl::RowCal64* cal64 = nullptr;
  float* calt32 = nullptr;           // [M] position t in [0, 1] of each bin in its node interval
  double* calt64 = nullptr;
  double* calB = nullptr;            // per interval: the window's weights as cubics in t [n-1][4][4]
  double* kcal = nullptr;            // per detector: K1 [ncal], K2 [ncal][ncal]
  int cal_j0[gwl::MAXNODE] = {};
  int64_t cal_kb[gwl::MAXNODE] = {};
  double cal_slope = 0.0;            // cycles of calibration phase per unit of ln f and node difference, at most
  std::vector<double> band_f;        // while a calibrated event is made: its band-limited rows' frequencies
  std::vector<int> band_seg;         //   and node intervals
  double df = 0.0;
  double gmst = 0.0;
  gwl_detector dets[GWL_MAX_DET] = {};
  gwl::EventGeom geom = {};
  void* slab = nullptr;              // the allocation that holds the tables and constants below
  void* cal_slab = nullptr;          // and the calibration model's
  void* tab64 = nullptr;             // RowF64<ndet>[M]
  void* tab32 = nullptr;             // RowMixed<ndet>[M]
  gwl::RowGradF32* g32 = nullptr;    // [M]
  gwl::RowGradF64* g64 = nullptr;    // [M]
  gwl::BandHead* bands = nullptr;    // band-limited rows, kept in tab64 and g64 after the bins (null: none)
  int nlev[2] = {0, 0};              // its levels in a float64 and a mixed-precision call
  int64_t M_loop = 0;                // rows that a typical point's loop walks (launch shapes)
  double* fgrid = nullptr;           // [M] grid frequencies (ISCO cut-off only)
  double* kcum = nullptr;            // [ndet][M + 1] running sums of the K_det terms (ISCO cut-off only)
  gwl::EventConst* ec = nullptr;     // device copy
  gwl::EventConst ech = {};          // host copy
};

namespace gwl {

// A launch whose chunks hold at most this many bins walks the bins: making a group's plan takes about 4 us
// in a small call, a chunk of 16 bins less (1,000 points on one detector and 4,017 bins: 13.9 us a
// call against 15.2 with plans; one point on three detectors and 16,225 bins, 32 bins a chunk: 22.7
// against 18.8 with plans).
constexpr int kBandMinChunk = 20;

constexpr int64_t kMaxBatch = (int64_t)1 << 30;

// Whether a call in precision p runs the mixed-precision bin loop on this event. A
// relative-binning event always runs the float64 loop: its few hundred edge terms are each the
// sum of hundreds of bins, and float32 roundings on them (the stored V_e, the hardware phasor,
// the products) do not average down below the 1e-3 bound on loud events.
inline bool use_mixed(const gwl_event_s* ev, gwl_precision p) { return p == GWL_MIXED && ev->M_full == 0; }

gwl_status fail(gwl_status st, const char* fmt, ...);
gwl_status hip_fail(hipError_t e, const char* what);
void clear_error();
gwl_status check_device(int dev);
gwl_status make_geom(const gwl_detector* dets, int ndet, double gmst, EventGeom& g);
size_t row64_bytes(int nd);
size_t row32_bytes(int nd);
// launch shape of a live-length call of capacity B
LoopShape live_shape(const gwl_event_s* ev, int64_t B, bool mixed);
// workspace of an evaluation launch: set-up rows [NCOEF][Bp] unless the kernel does the set-up,
// then workgroup partial sums [G][nz][Bp] for the gradient or when G > 1 (doubles), and npg
// completion counters for the value when G > 1
// (and, with the set-up kernel, a plan per point group)
size_t workspace_bytes(int64_t Bp, const LoopShape& sh, int nd, bool grad);
size_t workspace_counters(const LoopShape& sh, bool grad);

// launch shape of a call (autotuner cache, else a heuristic)
LoopShape choose_shape(const gwl_event_s* ev, int64_t B, bool mixed, bool grad);
// (M bins, of which a typical point's loop walks `rows` rows)
LoopShape heuristic_shape(int64_t B, int64_t M, int64_t rows, bool mixed, bool grad);
// whether a call takes its points in launch_order's order: on band-limited rows, from 16,384 points on
// or, where a row costs about twice as much (gradients, calibrated events), 8,192. The ordering takes
// 6 us; with it and without, three detectors and 8 s: values of 8,192 points 40.0 and 39.4 us, of
// 16,384 52.8 and 56.0, of 65,536 152 and 182; gradients of 16,384 86.7 and 96.1; calibrated gradients
// of 8,192 169 and 185
bool in_order(const gwl_event_s* ev, int64_t B, bool grad, int chunk);

// multi-event plans: build with an explicit chunk length (0 = heuristic) and queue order; the
// tuner's cached choice for a workload (chunk 0 and ascending order when none is cached)
gwl_status build_plan(const gwl_event* evs, int E, const int64_t* B_e, gwl_precision prec, int with_grad,
                      int chunk_req, bool descending, gwl_plan* out);
void choose_multi_shape(const gwl_event* evs, int E, const int64_t* B_e, bool mixed, bool grad, int* chunk,
                        bool* descending);
// fill theta[B][P] with valid parameter points (timing inputs; P >= 11, zeros past column 11)
hipError_t fill_theta(double* theta, int64_t B, hipStream_t s, int P = NPARAM);

// live (device, may be null): evaluate only the first *live of the B points
gwl_status run_logl(gwl_event ev, const double* theta, int64_t B, bool mixed, bool grad, const LoopShape& sh,
                    double* logl, double* gradout, hipStream_t s, const int64_t* live = nullptr);
// a call on a calibrated event (its own set-up, bin loop and epilogue kernels) in the workspace
// ws of ws_bytes bytes (at least call_workspace_bytes), which the caller owns
gwl_status run_calibrated(gwl_event ev, const double* theta, int64_t B, bool mixed, bool grad, double* logl,
                          double* gradout, hipStream_t s, void* ws, size_t ws_bytes);

// The event's workspace on stream s, grown to at least `bytes` and `ncnt` counters (zero when new) if
// needed. Growing is refused while s is capturing a graph (GWL_E_INVALID): the caller reserves it
// beforehand with gwl_event_reserve or an ordinary call of the same size.
gwl_status event_workspace(gwl_event ev, hipStream_t s, size_t bytes, size_t ncnt, void** out,
                           unsigned int** cnt = nullptr);
// Workspace bytes a single-event call of this kind needs.
size_t call_workspace_bytes(const gwl_event_s* ev, int64_t B, bool mixed, bool grad);
hipError_t enqueue_logl(gwl_event ev, const double* theta, int64_t B, bool mixed, bool grad, const LoopShape& sh,
                        double* ws, unsigned int* cnt, double* logl, double* gradout, hipStream_t s,
                        const int64_t* live = nullptr);

}  // namespace gwl
