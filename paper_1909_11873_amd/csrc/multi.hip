// Several events of uneven duration and batch size in one persistent launch, captured in a
// HIP graph (the batch axis of the paper's parallel prior sampling, section 3, extended over
// events).
//
// Work items are (64-point group of an event, four chunks of its plan's rows). The set-up of a group
// makes its plan (gwl_bands.h: the band-limited rows, or the bins, that its points walk), cuts it into
// chunks of about one length for all events, so that items cost about the same, and appends them to
// the queue; events are queued shortest first. A workgroup of the persistent kernel takes every
// gridDim-th item, a chunk to each of its wavefronts, adds the four sums in LDS and writes the item's
// partial sums, which a multi-event epilogue launch adds in chunk order (deterministic, whatever the
// queue's order). Every item and group stamps the device clock into a place of its own; the host takes an
// event's latency from them. The graph is: reset -> per-point set-up and queue for all events ->
// persistent loop -> epilogue for all events.
//
// What bounds it: the loop's float64 instructions. Queue tickets, completion counters and stamps were
// device-scope atomics on one address, which the dies take in turn at about 20 ns each: 12,500 of them
// held 12 float64 gradient events of 4 to 64 s (516,000 rows of 64 points) at 262 us. Items dealt by
// index and stamps in places of their own: 170 us; one item per workgroup instead of per wavefront keeps
// that and writes a quarter of the partial sums (the epilogue: 25 -> 16 us), and the 64-event
// mixed-precision workload takes 1.60 ms for 1.72.
#include <hip/hip_runtime.h>

#include <math.h>
#include <stddef.h>
#include <string.h>

#include <algorithm>
#include <numeric>
#include <vector>

#include "gwl_bands.h"
#include "gwl_bins.h"
#include "gwl_epilogue.h"
#include "gwl_runtime.h"
#include "gwl_setup.h"

using namespace gwl;

namespace gwl {

constexpr int MULTI_SETUP_WAVES = 4;  // wavefronts per group of 64 points in the set-up
constexpr int MULTI_EPI_BLOCK = 256;  // points per workgroup of the value's epilogue
// bins per chunk of a group that walks its bins, at least (an item has four): 12 float64 events whose
// points arrive all over the segment, mostly on bins: 3.20 ms at 1,536, 2.75 at 384
constexpr int MULTI_BIN_CHUNK = 384;
constexpr int MULTI_ROUND_ROWS = 96;
constexpr int MULTI_RED = 4;          // sums reduced per LDS pass

struct MultiEvDev {
  const void* tab64;       // RowF64<ND>: bins (or edges), then the band-limited rows
  const void* tab32;       // RowMixed<ND> [M]
  const void* gtab;        // RowGradF64 (adjoint basis, both precisions)
  const EventConst* ec;
  const BandHead* bands;   // null: every bin
  double* coef;            // [NCOEF][Bp]
  double* part;            // [nslot][NZ][Bp]
  int64_t Bp;
  int M, nslot, npg;       // nslot: most chunks that a group may have
  int f64;                 // 1: float64 loop on every row (every event of a float64 plan, and the
                           // relative-binning events of a mixed one)
  int rot;                 // 1: a uniform grid: the float64 loop rotates the detectors' phasors
  double step;             // the grid's spacing
};

// a group's plan also holds its number of items and its first item
constexpr int PLAN_ITEMS = PLAN_INTS - 1, PLAN_BASE = PLAN_INTS - 2;

struct MultiIODev {
  const double* theta;     // [B][11]
  double* logl;            // [B]
  double* grad;            // [B][11] or null
  int64_t B;
};

struct MultiCtl {
  unsigned int total;      // items in the queue
  unsigned int pad;
  unsigned long long t0;   // device clock at the start of the launch
};

__global__ void k_multi_reset(MultiCtl* __restrict__ ctl) {
  ctl->total = 0u;
  ctl->t0 = wall_clock64();
}

// device clock stamp (a calibrated event's completion)
__global__ void k_multi_stamp(unsigned long long* __restrict__ t) { *t = wall_clock64(); }

// Set-up rows and plan of one group per workgroup (as k_setup), and the group's items: chunks of
// about `chunk` rows, all appended at once. The items' order in the queue may differ from run to run
// with the workgroups' timing; their results do not.
template <int ND>
__global__ __launch_bounds__(MULTI_SETUP_WAVES * WAVE) void k_multi_setup(
    const MultiEvDev* __restrict__ evs, const EventGeom* __restrict__ geoms, const MultiIODev* __restrict__ io,
    const int2* __restrict__ grp, int mixed, int grad, int chunk, MultiCtl* __restrict__ ctl, int2* __restrict__ items,
    int* __restrict__ plans) {
  alignas(16) __shared__ double rows_s[NCOEF * WAVE];
  __shared__ BandLds bands_s;
  __shared__ int base_s;
  const int2 gp = grp[blockIdx.x];
  const MultiEvDev ev = evs[gp.x];
  const MultiIODev o = io[gp.x];
  const EventGeom geo = geoms[gp.x];
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / WAVE));
  const int lane = (int)(threadIdx.x % WAVE);
  const int64_t p = (int64_t)gp.y * WAVE + lane;
  const int64_t pc = p < o.B ? p : o.B - 1;
  BandPre pre;
  if (ev.bands) pre = band_fetch(ev.bands, w, lane);
  double* slopes_s = rows_s + CO_CR * WAVE;                // (these rows go to memory only)
  if (w < 2) setup_halves<ND>(w, lane, o.theta + pc * NPARAM, geo, ev.ec, rows_s);
  else if (ev.bands) band_load(ev.bands, slopes_s, 2 * WAVE);
  __syncthreads();
  if (w < 2) setup_rows_write<ND>(w, lane, rows_s, ev.ec, true, ev.coef, ev.Bp, p);
  if (ev.bands) {
    double a[NBASIS], T[ND];
#pragma unroll
    for (int m = 0; m < NBASIS; ++m) a[m] = rows_s[(CO_A + m) * WAVE + lane];
#pragma unroll
    for (int d = 0; d < ND; ++d) T[d] = rows_s[(CO_T + d) * WAVE + lane];
    if (!rows_in_range<ND>(a, T, ev.ec)) a[0] = __builtin_nan("");
    band_ranges<ND>(slopes_s, pre.nbrk, a, T, w, MULTI_SETUP_WAVES, lane, bands_s);
    __syncthreads();
    band_hold(ev.bands, pre, slopes_s, w, MULTI_SETUP_WAVES, lane, bands_s);
    __syncthreads();
    if (w != 0) return;
    band_plan(pre, slopes_s, float64_most(mixed && !ev.f64, grad != 0, false, ev.M), 1, lane, bands_s);
  } else {
    if (w != 0) return;
    if (lane == 0) {                                   // the bins as one piece
      bands_s.plan[0] = bands_s.plan[5] = ev.M;
      bands_s.plan[1] = 1;
      bands_s.plan[2] = ev.f64;
      bands_s.plan[4] = 0;
      bands_s.plan[6] = -1;
    }
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // LDS from the lanes that wrote it
  if (lane == 0) {
    const int rows = bands_s.plan[2] ? bands_s.plan[0] : ev.M;
    int n = (rows + WAVES_PER_BLOCK * chunk - 1) / (WAVES_PER_BLOCK * chunk);
    if (n > ev.nslot) n = ev.nslot;
    bands_s.plan[3] = (rows + WAVES_PER_BLOCK * n - 1) / (WAVES_PER_BLOCK * n);
    bands_s.plan[PLAN_ITEMS] = n;
    bands_s.plan[PLAN_BASE] = base_s = (int)atomicAdd(&ctl->total, (unsigned int)n);
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // LDS from the lanes that wrote it
  const int n = bands_s.plan[PLAN_ITEMS], base = base_s;
  for (int c = lane; c < n; c += WAVE) items[base + c] = make_int2((int)blockIdx.x, c);
  plans[(int64_t)blockIdx.x * PLAN_INTS + lane] = bands_s.plan[lane];
}

// Wavefronts per SIMD that the register budget must allow. Three detectors' mixed adjoint holds both
// loops: at four it spilled 168 bytes a lane (64 events: 1.69 ms, 1.60 at three); the float64 one
// spills 96 at four and still gains (12 events: 169 us, 180 at three).
template <int ND, bool MIXED, bool GRAD>
constexpr int multi_waves_per_eu() {
  return ND > 3 || (ND == 3 && MIXED && GRAD) ? 3 : 4;
}

// Persistent loop: one workgroup per item, its wavefronts on four consecutive chunks of the group's
// rows.
template <int ND, bool MIXED, bool GRAD>
__global__ __launch_bounds__(BLOCK, (multi_waves_per_eu<ND, MIXED, GRAD>())) void k_multi_bins(
    const MultiEvDev* __restrict__ evs, const MultiIODev* __restrict__ io, const int2* __restrict__ grp,
    const int2* __restrict__ items, const int* __restrict__ plans, const MultiCtl* __restrict__ ctl,
    unsigned long long* __restrict__ stamp) {
  constexpr int NZ = nz_of(ND, GRAD);
  __shared__ double2 tbl[PH_TBL];  // the float64 phasor table
  __shared__ double red[WAVES_PER_BLOCK - 1][MULTI_RED][WAVE];
  fill_phasor_table(tbl);
  __syncthreads();
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / WAVE));
  const int lane = threadIdx.x % WAVE;
  const int total = (int)__builtin_amdgcn_readfirstlane(ctl->total);
  for (int it = (int)blockIdx.x; it < total; it += (int)gridDim.x) {
    const int2 item = items[it];
    const int2 gp = grp[item.x];
    const int e = gp.x, c = item.y * WAVES_PER_BLOCK + w;
    const MultiEvDev ev = evs[e];
    const int* plan = plans + (int64_t)item.x * PLAN_INTS;
    const int64_t B = io[e].B;
    const int64_t p = (int64_t)gp.y * WAVE + lane;
    const int64_t pc = p < B ? p : B - 1;
    const bool f64path = plan[2] != 0;                 // scalar branch
    const int rows = f64path ? plan[0] : ev.M, q0 = c * plan[3];
    const int q1 = q0 + plan[3] < rows ? q0 + plan[3] : rows;   // none when q0 >= q1
    double tot[NZ];
#pragma unroll
    for (int z = 0; z < NZ; ++z) tot[z] = 0.0;
    double a[NBASIS], T[ND], crd[ND], cid[ND];
    load_coef<ND, double>(ev.coef, ev.Bp, pc, GRAD, a, T, crd, cid);
    if (!f64path) {
      if constexpr (MIXED) {
        float cr[ND], ci[ND];
        if constexpr (GRAD) {
          mixed_factors<ND>(ev.ec, crd, cid, cr, ci);
        } else {
#pragma unroll
          for (int d = 0; d < ND; ++d) cr[d] = ci[d] = 0.0f;
        }
        bin_loop_mixed<ND, GRAD>((const_as_ptr<RowMixed<ND>>)ev.tab32, (const_as_ptr<RowGradF64>)ev.gtab, q0, q1, a, T,
                                 cr, ci, tot);
        mixed_units<ND, GRAD>(ev.ec, tot);
      }
    } else {
      to_table_units<ND>(a, T);
      for_pieces(
          ev.bands, ev.step, q0, q1, [&](int i) { return plan[i]; },
          [&](int ka, int kb, double step) {
            if (ev.rot)
              bin_loop_f64_rot<ND, GRAD>((const_as_ptr<RowF64<ND>>)ev.tab64, (const_as_ptr<RowGradF64>)ev.gtab, ka, kb,
                                         a, T, crd, cid, tbl, step, tot);
            else
              bin_loop_f64<ND, GRAD>((const_as_ptr<RowF64<ND>>)ev.tab64, (const_as_ptr<RowGradF64>)ev.gtab, ka, kb, a,
                                     T, crd, cid, tbl, tot);
          });
    }
    global_as_ptr<double> part = (global_as_ptr<double>)ev.part;
    // the item's four sums, added in chunk order by the first wavefront
#pragma unroll
    for (int z0 = 0; z0 < NZ; z0 += MULTI_RED) {
      __syncthreads();
      if (w > 0) {
#pragma unroll
        for (int zz = 0; zz < MULTI_RED; ++zz)
          if (z0 + zz < NZ) red[w - 1][zz][lane] = tot[z0 + zz];
      }
      __syncthreads();
      if (w == 0) {
#pragma unroll
        for (int zz = 0; zz < MULTI_RED; ++zz)
          if (z0 + zz < NZ) {
#pragma unroll
            for (int v = 0; v < WAVES_PER_BLOCK - 1; ++v) tot[z0 + zz] += red[v][zz][lane];
            part[((int64_t)item.y * NZ + z0 + zz) * ev.Bp + p] = tot[z0 + zz];
          }
      }
    }
    if (threadIdx.x == 0) stamp[it] = wall_clock64();
  }
}

// A group's clock stamps: its last item's, and its epilogue's.
__device__ inline void group_stamps(const unsigned long long* __restrict__ stamp, int n, int lane,
                                    unsigned long long* __restrict__ out) {
  unsigned long long t = 0;
  for (int c = lane; c < n; c += WAVE) t = stamp[c] > t ? stamp[c] : t;
#pragma unroll
  for (int off = WAVE / 2; off > 0; off >>= 1) {
    const unsigned long long o = __shfl_xor(t, off);
    t = o > t ? o : t;
  }
  if (lane == 0) {
    out[0] = t;
    out[1] = wall_clock64();
  }
}

// The gradient's epilogue: one workgroup of four wavefronts per group, as k_epilogue_grad.
constexpr int MULTI_EPG_WAVES = 4;
template <int ND>
__global__ __launch_bounds__(MULTI_EPG_WAVES * WAVE) void k_multi_epilogue_grad(
    const MultiEvDev* __restrict__ evs, const EventGeom* __restrict__ geoms, const MultiIODev* __restrict__ io,
    const int2* __restrict__ grp, const int* __restrict__ plans, const unsigned long long* __restrict__ stamp,
    unsigned long long* __restrict__ gstamp) {
  constexpr int NZ = nz_of(ND, true);
  __shared__ double acc_s[NZ][WAVE];
  __shared__ double xs[GRAD_LDS][WAVE];
  const int2 gp = grp[blockIdx.x];
  const MultiEvDev ev = evs[gp.x];
  const MultiIODev o = io[gp.x];
  const int n = plans[(int64_t)blockIdx.x * PLAN_INTS + PLAN_ITEMS];
  const int base = plans[(int64_t)blockIdx.x * PLAN_INTS + PLAN_BASE];
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / WAVE));
  const int lane = (int)(threadIdx.x % WAVE);
  const int64_t p = (int64_t)gp.y * WAVE + lane;
  const int64_t pc = p < o.B ? p : o.B - 1;
  gather_share<NZ, MULTI_EPG_WAVES>(ev.part, n, ev.Bp, p, w, lane, acc_s);
  double th[NPARAM];
#pragma unroll
  for (int i = 0; i < NPARAM; ++i) th[i] = o.theta[pc * NPARAM + i];
  __syncthreads();
  GradParts<ND> r;
  gradient_parts<ND>(w, lane, acc_s, th, geoms[gp.x], xs, r);
  __syncthreads();
  if (w < 2 && p < o.B) {
    double K[ND];
#pragma unroll
    for (int d = 0; d < ND; ++d) K[d] = ev.ec->K[d];
    gradient_finish<ND>(w, lane, th, K, xs, r, o.logl + p, o.grad + p * NPARAM);
  }
  if (w == 3) group_stamps(stamp + base, n, lane, gstamp + 2 * (int64_t)blockIdx.x);
}

// The value's epilogue: a thread per point, four groups per workgroup.
template <int ND>
__global__ __launch_bounds__(MULTI_EPI_BLOCK) void k_multi_epilogue(
    const MultiEvDev* __restrict__ evs, const MultiIODev* __restrict__ io, const int2* __restrict__ grp, int ngrp,
    const int* __restrict__ plans, const unsigned long long* __restrict__ stamp,
    unsigned long long* __restrict__ gstamp) {
  constexpr int NZ = nz_of(ND, false);
  const int g = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * (MULTI_EPI_BLOCK / WAVE) + threadIdx.x / WAVE));
  if (g < ngrp) {
    const int2 gp = grp[g];
    const MultiEvDev ev = evs[gp.x];
    const MultiIODev o = io[gp.x];
    const int64_t p = (int64_t)gp.y * WAVE + threadIdx.x % WAVE;
    if (p < o.B) {
      double acc[NZ];
      gather<NZ>(ev.part, plans[(int64_t)g * PLAN_INTS + PLAN_ITEMS], ev.Bp, p, acc);
      o.logl[p] = epilogue_value_rows<ND, NZ>(acc, ev.coef, ev.Bp, p, *ev.ec, 1.0);
    }
    const int* plan = plans + (int64_t)g * PLAN_INTS;
    group_stamps(stamp + plan[PLAN_BASE], plan[PLAN_ITEMS], (int)(threadIdx.x % WAVE), gstamp + 2 * (int64_t)g);
  }
}

}  // namespace gwl

struct gwl_plan_s {
  int device = 0;
  int E = 0, nd = 0;
  bool mixed = false, grad = false;
  std::vector<int64_t> B;
  std::vector<gwl_event> evs;  // the events (event order)
  std::vector<int> cal;        // calibrated events (event index): their own kernels, after the graph
  std::vector<int> order;      // queue position -> event index
  int total = 0, grid = 0, ngrp = 0, chunk = 0;  // total: items when every group walks a typical one's rows
  bool descending = false;     // queue order: events by descending work instead of ascending
  double clock_khz = 0.0;
  gwl::MultiEvDev* d_evs = nullptr;   // in queue order
  gwl::EventGeom* d_geoms = nullptr;  // in queue order
  gwl::MultiIODev* d_io = nullptr;    // in queue order
  gwl::MultiIODev* h_io = nullptr;    // pinned host staging
  int2* d_grp = nullptr;              // [ngrp]: event (queue index), point group
  int2* d_items = nullptr;            // the queue: group, chunk
  int* d_plans = nullptr;             // [ngrp][PLAN_INTS]
  void* d_ctl = nullptr;              // MultiCtl, tev[E] (calibrated events), gstamp[ngrp][2], stamp[items]
  unsigned long long* h_stamps = nullptr;  // pinned: the control block without the items' stamps
  double* ws = nullptr;
  hipStream_t cap = nullptr;
  hipGraph_t graph = nullptr;
  hipGraphExec_t exec = nullptr;
  hipEvent_t io_done = nullptr;
  // calibrated events run on side streams (default priority) after the graph, the calibrated
  // events in turn, each stream in a workspace of the plan's own sized for its largest event
  static constexpr int kCalStreams = 4;
  hipStream_t cal_s[kCalStreams] = {};
  void* cal_ws[kCalStreams] = {};
  size_t cal_ws_bytes[kCalStreams] = {};
  hipEvent_t cal_fork = nullptr;
  hipEvent_t cal_join[kCalStreams] = {};
};

namespace {

// Set to false to switch the multi-event plan off.
constexpr bool kMultiEnabled = true;

// the control block: the calibrated events' stamps, the groups' (last item, epilogue), the items'
constexpr size_t kTevOffset = sizeof(gwl::MultiCtl);
size_t gstamp_offset(int E) { return kTevOffset + sizeof(unsigned long long) * (size_t)E; }
size_t stamp_offset(int E, int ngrp) { return gstamp_offset(E) + 2 * sizeof(unsigned long long) * (size_t)ngrp; }

// precision of calibrated event e's own kernels in plan pl (as its single call would take)
bool mixed_cal(const gwl_plan_s* pl, int e) { return pl->mixed && use_mixed(pl->evs[e], GWL_MIXED); }

void plan_free(gwl_plan pl) {
  if (!pl) return;
  if (pl->exec) (void)hipGraphExecDestroy(pl->exec);
  if (pl->graph) (void)hipGraphDestroy(pl->graph);
  if (pl->cap) (void)hipStreamDestroy(pl->cap);
  if (pl->io_done) (void)hipEventDestroy(pl->io_done);
  for (int i = 0; i < gwl_plan_s::kCalStreams; ++i) {
    if (pl->cal_s[i]) (void)hipStreamDestroy(pl->cal_s[i]);
    if (pl->cal_join[i]) (void)hipEventDestroy(pl->cal_join[i]);
    if (pl->cal_ws[i]) (void)hipFree(pl->cal_ws[i]);
  }
  if (pl->cal_fork) (void)hipEventDestroy(pl->cal_fork);
  if (pl->d_evs) (void)hipFree(pl->d_evs);
  if (pl->d_geoms) (void)hipFree(pl->d_geoms);
  if (pl->d_io) (void)hipFree(pl->d_io);
  if (pl->d_grp) (void)hipFree(pl->d_grp);
  if (pl->d_items) (void)hipFree(pl->d_items);
  if (pl->d_plans) (void)hipFree(pl->d_plans);
  if (pl->d_ctl) (void)hipFree(pl->d_ctl);
  if (pl->ws) (void)hipFree(pl->ws);
  if (pl->h_io) (void)hipHostFree(pl->h_io);
  if (pl->h_stamps) (void)hipHostFree(pl->h_stamps);
  delete pl;
}

template <int ND>
hipError_t enqueue_multi_nd(gwl_plan pl, hipStream_t s) {
  const int E = pl->E;
  unsigned char* ctl = (unsigned char*)pl->d_ctl;
  gwl::MultiCtl* c = (gwl::MultiCtl*)ctl;
  unsigned long long* gstamp = (unsigned long long*)(ctl + gstamp_offset(E));
  unsigned long long* stamp = (unsigned long long*)(ctl + stamp_offset(E, pl->ngrp));
  const gwl::MultiEvDev* evs = pl->d_evs;
  const gwl::EventGeom* geoms = pl->d_geoms;
  const gwl::MultiIODev* io = pl->d_io;
  const int2* grp = pl->d_grp;
  hipLaunchKernelGGL(gwl::k_multi_reset, dim3(1), dim3(1), 0, s, c);
  if (pl->ngrp == 0) return hipGetLastError();   // no point outside calibrated events: only the reset
  hipLaunchKernelGGL(gwl::k_multi_setup<ND>, dim3(pl->ngrp), dim3(gwl::MULTI_SETUP_WAVES * gwl::WAVE), 0, s, evs, geoms,
                     io, grp, pl->mixed ? 1 : 0, pl->grad ? 1 : 0, pl->chunk, c, pl->d_items, pl->d_plans);
#define GWL_MB(MX, GR)                                                                                         \
  hipLaunchKernelGGL((gwl::k_multi_bins<ND, MX, GR>), dim3(pl->grid), dim3(gwl::BLOCK), 0, s, evs, io, grp,    \
                     (const int2*)pl->d_items, (const int*)pl->d_plans, (const gwl::MultiCtl*)c, stamp)
  if (pl->mixed) {
    if (pl->grad) GWL_MB(true, true); else GWL_MB(true, false);
  } else {
    if (pl->grad) GWL_MB(false, true); else GWL_MB(false, false);
  }
#undef GWL_MB
  if (pl->grad) {
    hipLaunchKernelGGL(gwl::k_multi_epilogue_grad<ND>, dim3(pl->ngrp), dim3(gwl::MULTI_EPG_WAVES * gwl::WAVE), 0, s, evs,
                       geoms, io, grp, (const int*)pl->d_plans, (const unsigned long long*)stamp, gstamp);
  } else {
    constexpr int per = gwl::MULTI_EPI_BLOCK / gwl::WAVE;
    hipLaunchKernelGGL(gwl::k_multi_epilogue<ND>, dim3((pl->ngrp + per - 1) / per), dim3(gwl::MULTI_EPI_BLOCK), 0, s,
                       evs, io, grp, pl->ngrp, (const int*)pl->d_plans, (const unsigned long long*)stamp, gstamp);
  }
  return hipGetLastError();
}

hipError_t enqueue_multi(gwl_plan pl, hipStream_t s) {
  switch (pl->nd) {
    case 1: return enqueue_multi_nd<1>(pl, s);
    case 2: return enqueue_multi_nd<2>(pl, s);
    case 3: return enqueue_multi_nd<3>(pl, s);
    case 4: return enqueue_multi_nd<4>(pl, s);
  }
  return hipErrorInvalidValue;
}

template <int ND>
hipError_t occupancy_nd(bool mixed, bool grad, int* nblk) {
#define GWL_OCC(MX, GR) return hipOccupancyMaxActiveBlocksPerMultiprocessor(nblk, gwl::k_multi_bins<ND, MX, GR>, gwl::BLOCK, 0)
  if (mixed) {
    if (grad) GWL_OCC(true, true); else GWL_OCC(true, false);
  }
  if (grad) GWL_OCC(false, true); else GWL_OCC(false, false);
#undef GWL_OCC
}

hipError_t occupancy(int nd, bool mixed, bool grad, int* nblk) {
  switch (nd) {
    case 1: return occupancy_nd<1>(mixed, grad, nblk);
    case 2: return occupancy_nd<2>(mixed, grad, nblk);
    case 3: return occupancy_nd<3>(mixed, grad, nblk);
    case 4: return occupancy_nd<4>(mixed, grad, nblk);
  }
  return hipErrorInvalidValue;
}

}  // namespace

namespace gwl {

// Build a plan with a given chunk length (0: the heuristic) and queue order.
gwl_status build_plan(const gwl_event* evs, int E, const int64_t* B_e, gwl_precision prec, int with_grad,
                      int chunk_req, bool descending, gwl_plan* out) {
  if (!out) return fail(GWL_E_INVALID, "out is null");
  *out = nullptr;
  if (!evs || !B_e) return fail(GWL_E_INVALID, "evs and B_e must be host arrays");
  if (E < 1 || E > 4096) return fail(GWL_E_SHAPE, "E=%d outside [1, 4096]", E);
  if (prec != GWL_FP64 && prec != GWL_MIXED) return fail(GWL_E_INVALID, "unknown precision %d", (int)prec);
  const int nd = evs[0] ? evs[0]->ndet : 0;
  for (int e = 0; e < E; ++e) {
    if (!evs[e]) return fail(GWL_E_INVALID, "event %d is null", e);
    if (evs[e]->ndet != nd) return fail(GWL_E_UNSUPPORTED, "events must share one detector count");
    if (evs[e]->ech.isco) return fail(GWL_E_UNSUPPORTED, "event %d has the ISCO cut-off: not in multi-event plans", e);
    if (evs[e]->device != evs[0]->device) return fail(GWL_E_INVALID, "events must live on one device");
    if (B_e[e] < 0 || B_e[e] > kMaxBatch) return fail(GWL_E_SHAPE, "B_e[%d]=%lld out of range", e, (long long)B_e[e]);
  }
  gwl_status st = check_device(evs[0]->device);
  if (st != GWL_OK) return st;
  if (!kMultiEnabled)
    return fail(GWL_E_UNSUPPORTED, "the persistent multi-event launch is switched off");

  gwl_plan pl = new (std::nothrow) gwl_plan_s();
  if (!pl) return fail(GWL_E_NOMEM, "host allocation failed");
  pl->device = evs[0]->device;
  pl->E = E;
  pl->nd = nd;
  pl->mixed = prec == GWL_MIXED;
  pl->grad = with_grad != 0;
  pl->B.assign(B_e, B_e + E);
  pl->evs.assign(evs, evs + E);
  for (int e = 0; e < E; ++e)
    if (evs[e]->ncal > 0) pl->cal.push_back(e);

  hipError_t err = hipSuccess;
  int occ = 0, ncu = 0, clk = 0;
  err = occupancy(nd, pl->mixed, pl->grad, &occ);
  if (err == hipSuccess) err = hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, pl->device);
  if (err == hipSuccess) err = hipDeviceGetAttribute(&clk, hipDeviceAttributeWallClockRate, pl->device);
  if (err != hipSuccess) {
    plan_free(pl);
    return hip_fail(err, "device query");
  }
  if (occ < 1) occ = 1;
  pl->grid = occ * ncu;
  pl->clock_khz = (double)clk;
  auto items_for = [&](int chunk) {
    int64_t n = 0;
    for (int e = 0; e < E; ++e) {
      if (B_e[e] == 0 || evs[e]->ncal > 0) continue;
      const int64_t len = (int64_t)WAVES_PER_BLOCK * chunk;
      n += ((B_e[e] + WAVE - 1) / WAVE) * ((evs[e]->M_loop + len - 1) / len);
    }
    return n;
  };
  // one chunk length for all events: the shortest with which the items of typical groups fill a whole
  // number of rounds of the resident workgroups to nineteen twentieths at most, as many rounds (up to
  // four) as keep it near MULTI_ROUND_ROWS, and 512 rows at most. On 12 events of 4 to 64 s in float64:
  // 168 to 171 us at 48 to 96 rows, 185 at 128, 247 at 384; on 64 events 1.55 ms at 256, 1.60 at 4096
  auto shortest = [&](int64_t rounds) {
    int c = 32;
    while (c < 512 && 20 * items_for(c) > 19 * rounds * pl->grid) c += 8;
    return c;
  };
  int chunk = shortest(1);
  if (chunk > MULTI_ROUND_ROWS) chunk = shortest(std::min(4, (chunk + MULTI_ROUND_ROWS - 1) / MULTI_ROUND_ROWS));
  if (chunk_req > 0) chunk = chunk_req;
  const int64_t total = items_for(chunk);
  // most chunks of a group of event e: enough for half as many rows again as a typical group's, and for
  // its bins in chunks of MULTI_BIN_CHUNK
  auto slots = [&](const gwl_event ev) {
    const int64_t len = (int64_t)WAVES_PER_BLOCK * chunk, blen = (int64_t)WAVES_PER_BLOCK * std::max(chunk, MULTI_BIN_CHUNK);
    const int64_t rows = std::min<int64_t>((ev->M_loop + ev->M_loop / 2 + len - 1) / len, (ev->M + len - 1) / len);
    const int64_t bins = (ev->M + blen - 1) / blen;
    return std::max<int64_t>(1, std::max(rows, bins));
  };
  int64_t capacity = 0, ngroups = 0;
  for (int e = 0; e < E; ++e) {
    if (evs[e]->ncal > 0) continue;
    const int64_t n = (B_e[e] + WAVE - 1) / WAVE;
    ngroups += n;
    capacity += n * slots(evs[e]);
  }
  if (total > ((int64_t)1 << 30) || capacity > ((int64_t)1 << 30)) {
    plan_free(pl);
    return fail(GWL_E_SHAPE, "too many work items (%lld)", (long long)total);
  }
  pl->chunk = chunk;
  pl->total = (int)total;

  // queue order: events by ascending (or descending) work, ties by index
  pl->descending = descending;
  pl->order.resize(E);
  std::iota(pl->order.begin(), pl->order.end(), 0);
  std::stable_sort(pl->order.begin(), pl->order.end(), [&](int a, int b) {
    const double wa = (double)B_e[a] * (double)evs[a]->M_loop, wb = (double)B_e[b] * (double)evs[b]->M_loop;
    return descending ? wa > wb : wa < wb;
  });

  // workspace and device tables
  const int NZ = nz_of(nd, pl->grad);
  std::vector<MultiEvDev> hev(E);
  std::vector<EventGeom> hgeo(E);
  std::vector<int2> grp;
  grp.reserve((size_t)ngroups);
  size_t ws_doubles = 0;
  for (int q = 0; q < E; ++q) {
    const int e = pl->order[q];
    const gwl_event ev = evs[e];
    MultiEvDev& d = hev[q];
    memset(&d, 0, sizeof d);
    const int64_t B = evs[e]->ncal > 0 ? 0 : B_e[e];   // calibrated events are not in the queue
    d.npg = (int)((B + WAVE - 1) / WAVE);
    d.Bp = (int64_t)d.npg * WAVE;
    d.M = (int)ev->M;
    d.nslot = (int)slots(ev);
    d.f64 = use_mixed(ev, prec) ? 0 : 1;
    d.rot = ev->ech.uniform != 0 ? 1 : 0;
    d.step = ev->ech.grid_df;
    d.tab64 = ev->tab64;
    d.tab32 = ev->tab32;
    d.gtab = ev->g64;
    d.ec = ev->ec;
    d.bands = ev->bands;
    ws_doubles += (size_t)NCOEF * d.Bp + (size_t)d.nslot * NZ * d.Bp;
    hgeo[q] = ev->geom;
    for (int pg = 0; pg < d.npg; ++pg) grp.push_back(make_int2(q, pg));
  }
  pl->ngrp = (int)grp.size();
  err = hipMalloc((void**)&pl->ws, sizeof(double) * (ws_doubles > 0 ? ws_doubles : 1));
  size_t off = 0;
  for (int q = 0; q < E; ++q) {
    MultiEvDev& d = hev[q];
    d.coef = pl->ws + off;
    off += (size_t)NCOEF * d.Bp;
    d.part = pl->ws + off;
    off += (size_t)d.nslot * NZ * d.Bp;
  }
  if (err == hipSuccess) err = hipMalloc((void**)&pl->d_evs, sizeof(MultiEvDev) * E);
  if (err == hipSuccess) err = hipMalloc((void**)&pl->d_geoms, sizeof(EventGeom) * E);
  if (err == hipSuccess) err = hipMalloc((void**)&pl->d_io, sizeof(MultiIODev) * E);
  if (err == hipSuccess) err = hipMalloc((void**)&pl->d_grp, sizeof(int2) * (grp.empty() ? 1 : grp.size()));
  if (err == hipSuccess) err = hipMalloc((void**)&pl->d_items, sizeof(int2) * (size_t)(capacity > 0 ? capacity : 1));
  if (err == hipSuccess) err = hipMalloc((void**)&pl->d_plans, sizeof(int) * PLAN_INTS * (grp.empty() ? 1 : grp.size()));
  if (err == hipSuccess) err = hipMalloc(&pl->d_ctl, stamp_offset(E, pl->ngrp) + sizeof(unsigned long long) * (size_t)(capacity > 0 ? capacity : 1));
  if (err == hipSuccess) err = hipHostMalloc((void**)&pl->h_io, sizeof(MultiIODev) * E, hipHostMallocDefault);
  if (err == hipSuccess)
    err = hipHostMalloc((void**)&pl->h_stamps, stamp_offset(E, pl->ngrp), hipHostMallocDefault);
  if (err == hipSuccess) err = hipMemcpy(pl->d_evs, hev.data(), sizeof(MultiEvDev) * E, hipMemcpyHostToDevice);
  if (err == hipSuccess) err = hipMemcpy(pl->d_geoms, hgeo.data(), sizeof(EventGeom) * E, hipMemcpyHostToDevice);
  if (err == hipSuccess && !grp.empty())
    err = hipMemcpy(pl->d_grp, grp.data(), sizeof(int2) * grp.size(), hipMemcpyHostToDevice);
  if (err == hipSuccess) {
    memset(pl->h_io, 0, sizeof(MultiIODev) * E);
    err = hipMemcpy(pl->d_io, pl->h_io, sizeof(MultiIODev) * E, hipMemcpyHostToDevice);
  }
  if (err == hipSuccess) err = hipEventCreateWithFlags(&pl->io_done, hipEventDisableTiming);
  if (err == hipSuccess) err = hipStreamCreateWithFlags(&pl->cap, hipStreamNonBlocking);
  if (!pl->cal.empty()) {
    if (err == hipSuccess) err = hipEventCreateWithFlags(&pl->cal_fork, hipEventDisableTiming);
    for (int i = 0; i < gwl_plan_s::kCalStreams && err == hipSuccess; ++i) {
      err = hipStreamCreateWithFlags(&pl->cal_s[i], hipStreamNonBlocking);
      if (err == hipSuccess) err = hipEventCreateWithFlags(&pl->cal_join[i], hipEventDisableTiming);
    }
    int next = 0;
    for (int e : pl->cal) {
      if (pl->B[e] == 0) continue;
      const int i = next++ % gwl_plan_s::kCalStreams;
      pl->cal_ws_bytes[i] = std::max(pl->cal_ws_bytes[i],
                                     call_workspace_bytes(pl->evs[e], pl->B[e], mixed_cal(pl, e), pl->grad));
    }
    for (int i = 0; i < gwl_plan_s::kCalStreams && err == hipSuccess; ++i)
      if (pl->cal_ws_bytes[i] > 0) err = hipMalloc(&pl->cal_ws[i], pl->cal_ws_bytes[i]);
  }
  // capture the whole evaluation once
  if (err == hipSuccess) err = hipStreamBeginCapture(pl->cap, hipStreamCaptureModeThreadLocal);
  if (err == hipSuccess) {
    hipError_t e1 = enqueue_multi(pl, pl->cap);
    hipError_t e2 = hipStreamEndCapture(pl->cap, &pl->graph);
    err = e1 != hipSuccess ? e1 : e2;
  }
  if (err == hipSuccess) err = hipGraphInstantiate(&pl->exec, pl->graph, nullptr, nullptr, 0);
  if (err != hipSuccess) {
    plan_free(pl);
    return hip_fail(err, "multi-event plan");
  }
  *out = pl;
  return GWL_OK;
}

}  // namespace gwl

extern "C" {

gwl_status gwl_multi_plan_create(const gwl_event* evs, int E, const int64_t* B_e, gwl_precision prec, int with_grad,
                                 gwl_plan* out) {
  clear_error();
  int chunk = 0;
  bool desc = false;
  if (evs && B_e && E >= 1 && E <= 4096) {
    bool ok = true;
    for (int e = 0; e < E; ++e) ok &= evs[e] != nullptr;
    if (ok) choose_multi_shape(evs, E, B_e, prec == GWL_MIXED, with_grad != 0, &chunk, &desc);
  }
  return build_plan(evs, E, B_e, prec, with_grad, chunk, desc, out);
}

gwl_status gwl_multi_plan_create_order(const gwl_event* evs, int E, const int64_t* B_e, gwl_precision prec,
                                       int with_grad, int order, gwl_plan* out) {
  clear_error();
  if (order < 0 || order > 2) return fail(GWL_E_INVALID, "order must be 0 (tuned), 1 (ascending) or 2 (descending)");
  int chunk = 0;
  bool desc = false;
  if (evs && B_e && E >= 1 && E <= 4096) {
    bool ok = true;
    for (int e = 0; e < E; ++e) ok &= evs[e] != nullptr;
    if (ok) choose_multi_shape(evs, E, B_e, prec == GWL_MIXED, with_grad != 0, &chunk, &desc);
  }
  if (order == 1) desc = false;
  if (order == 2) desc = true;
  return build_plan(evs, E, B_e, prec, with_grad, chunk, desc, out);
}

gwl_status gwl_plan_info(gwl_plan pl, int* chunk, int* descending, int64_t* items) {
  clear_error();
  if (!pl) return fail(GWL_E_INVALID, "plan is null");
  if (chunk) *chunk = pl->chunk;
  if (descending) *descending = pl->descending ? 1 : 0;
  if (items) *items = pl->total;
  return GWL_OK;
}

gwl_status gwl_multi_launch(gwl_plan pl, const double* const* theta, double* const* logl, double* const* grad,
                            double* event_latency_us, void* stream) {
  clear_error();
  if (!pl) return fail(GWL_E_INVALID, "plan is null");
  if (!theta || !logl) return fail(GWL_E_INVALID, "theta and logl must be host arrays of device pointers");
  if (pl->grad && !grad) return fail(GWL_E_INVALID, "the plan computes gradients: grad must be given");
  for (int e = 0; e < pl->E; ++e) {
    if (pl->B[e] == 0) continue;
    if (!theta[e] || !logl[e] || (pl->grad && !grad[e]))
      return fail(GWL_E_INVALID, "event %d: null device pointer", e);
  }
  gwl_status st = check_device(pl->device);
  if (st != GWL_OK) return st;
  hipStream_t s = (hipStream_t)stream;
  // the staging buffer is reused: wait until the previous upload has been consumed
  hipError_t err = hipEventSynchronize(pl->io_done);
  if (err != hipSuccess) return hip_fail(err, "plan staging");
  for (int q = 0; q < pl->E; ++q) {
    const int e = pl->order[q];
    pl->h_io[q].theta = theta[e];
    pl->h_io[q].logl = logl[e];
    pl->h_io[q].grad = pl->grad ? grad[e] : nullptr;
    pl->h_io[q].B = pl->evs[e]->ncal > 0 ? 0 : pl->B[e];
  }
  err = hipMemcpyAsync(pl->d_io, pl->h_io, sizeof(MultiIODev) * pl->E, hipMemcpyHostToDevice, s);
  if (err == hipSuccess) err = hipEventRecord(pl->io_done, s);
  if (err == hipSuccess) err = hipGraphLaunch(pl->exec, s);
  if (err != hipSuccess) return hip_fail(err, "multi-event launch");
  // calibrated events: their own set-up, bin-loop and epilogue kernels, each followed by a clock
  // stamp in the event's slot, dealt in turn to the plan's side streams after the graph (one small
  // event at a time leaves most of the chip idle); the caller's stream then waits for them all
  unsigned long long* tev_dev = (unsigned long long*)((unsigned char*)pl->d_ctl + kTevOffset);
  if (!pl->cal.empty()) {
    constexpr int NS = gwl_plan_s::kCalStreams;
    err = hipEventRecord(pl->cal_fork, s);
    for (int i = 0; i < NS && err == hipSuccess; ++i) err = hipStreamWaitEvent(pl->cal_s[i], pl->cal_fork, 0);
    if (err != hipSuccess) return hip_fail(err, "multi-event launch");
    int next = 0;
    for (int e : pl->cal) {
      if (pl->B[e] == 0) continue;
      const int i = next++ % NS;
      hipStream_t cs = pl->cal_s[i];
      st = run_calibrated(pl->evs[e], theta[e], pl->B[e], mixed_cal(pl, e), pl->grad, logl[e],
                          pl->grad ? grad[e] : nullptr, cs, pl->cal_ws[i], pl->cal_ws_bytes[i]);
      if (st != GWL_OK) break;
      int q = 0;
      while (pl->order[q] != e) ++q;
      hipLaunchKernelGGL(k_multi_stamp, dim3(1), dim3(1), 0, cs, tev_dev + q);
      err = hipGetLastError();
      if (err != hipSuccess) break;
    }
    // join, also after a failure, so that nothing queued on a side stream outlives the call's order
    hipError_t jerr = hipSuccess;
    for (int i = 0; i < NS; ++i) {
      hipError_t e1 = hipEventRecord(pl->cal_join[i], pl->cal_s[i]);
      if (e1 == hipSuccess) e1 = hipStreamWaitEvent(s, pl->cal_join[i], 0);
      if (e1 != hipSuccess && jerr == hipSuccess) jerr = e1;
    }
    if (st != GWL_OK) return st;
    if (err != hipSuccess) return hip_fail(err, "multi-event launch");
    if (jerr != hipSuccess) return hip_fail(jerr, "multi-event launch");
  }
  if (event_latency_us) {
    err = hipMemcpyAsync(pl->h_stamps, pl->d_ctl, stamp_offset(pl->E, pl->ngrp), hipMemcpyDeviceToHost, s);
    if (err == hipSuccess) err = hipStreamSynchronize(s);
    if (err != hipSuccess) return hip_fail(err, "latency read-back");
    const unsigned char* h = (const unsigned char*)pl->h_stamps;
    const unsigned long long t0 = ((const gwl::MultiCtl*)h)->t0;
    const unsigned long long* tcal = (const unsigned long long*)(h + kTevOffset);
    const unsigned long long* gs = (const unsigned long long*)(h + gstamp_offset(pl->E));
    // each event's last item, the last item and the end of the epilogue
    std::vector<unsigned long long> tev(tcal, tcal + pl->E);
    unsigned long long tbins = t0, tend = t0;
    int g = 0;
    for (int q = 0; q < pl->E; ++q) {
      const int e = pl->order[q];
      if (pl->evs[e]->ncal > 0) continue;
      tev[q] = t0;
      for (const int g1 = g + (int)((pl->B[e] + WAVE - 1) / WAVE); g < g1; ++g) {
        tev[q] = std::max(tev[q], gs[2 * g]);
        tend = std::max(tend, gs[2 * g + 1]);
      }
      tbins = std::max(tbins, tev[q]);
    }
    // an event's results exist once its last item is done and the final epilogue launch has run
    const double epi_us = tend > tbins ? (double)(tend - tbins) * 1e3 / pl->clock_khz : 0.0;
    for (int q = 0; q < pl->E; ++q) {
      const int e = pl->order[q];
      const double extra = pl->evs[e]->ncal > 0 ? 0.0 : epi_us;   // calibrated: stamped after its epilogue
      event_latency_us[e] = pl->B[e] == 0 ? 0.0 : (double)(tev[q] - t0) * 1e3 / pl->clock_khz + extra;
    }
  }
  return GWL_OK;
}

gwl_status gwl_plan_destroy(gwl_plan pl) {
  plan_free(pl);
  return GWL_OK;
}

}  // extern "C"
