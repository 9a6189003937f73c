// Detector calibration model (paper section 2, "Models and parameter spaces": amplitude and
// phase corrections at frequency nodes, ten per detector): the calibrated model is
//   h_cal,det(f) = h_det(f) (1 + dA_det(f)) exp(i dphi_det(f)),
// dA and dphi cubic Catmull-Rom splines in ln f through the node values (theta columns
// 11 + 2 n det .. : n amplitude values, then n phase values in radians).
//
// The bin loop is the ordinary one with one more complex factor per (point, detector, bin):
// the spline value is a cubic in the bin's position within its node interval, its coefficients formed from
// the point's four window node values when the walk enters the interval (VGPRs; a chunk may cross several
// intervals); the four-term weights of the same cubic (RowCal, wave-uniform) serve the adjoint's node moments.
// <h_cal|h_cal> needs no per-bin work: with K_k = 4 df f_k^-7/3 / S_k,
//   sum_k K_k (1 + dA_k)^2 = K + 2 alpha.K1 + alpha.K2.alpha,
// K1_j = sum_k K_k w_kj and K2_jl = sum_k K_k w_kj w_kl computed once per event (alpha the
// amplitude node values, w_kj the spline weight of node j at bin k).
//
// Adjoint: besides the uncalibrated moments (with w = u p replaced by the calibrated product),
// per detector and window node i the sums sum_k w_ki Re(c q_k) (amplitude) and
// sum_k w_ki Im(c w_cal,k) (phase), q = u p exp(i dphi), w_cal = (1 + dA) q.
#include <hip/hip_runtime.h>

#include "gwl_bands.h"
#include "gwl_bins.h"
#include "gwl_common.h"
#include "gwl_device.h"
#include "gwl_epilogue.h"
#include "gwl_launch.h"
#include "gwl_setup.h"

namespace gwl {

// Set-up of a calibrated call: the point model's rows as k_setup writes them (two wavefronts, one
// per half of the model), and the calibration node values turned from theta's columns 11.. into
// rows calc [ncal][Bp], two more wavefronts copying half of them each; every row of a point with a
// non-finite node value is NaN. With band-limited rows the four bound the group's arrival times as k_setup's
// do, widened by the calibration phase: over a node interval's rows the spline's slope per node spacing is at
// most cal_slope (gwl_bands.h) times the largest difference of neighbouring node values.
constexpr int SETUP_CAL_WAVES = 4;
template <int ND>
__global__ __launch_bounds__(SETUP_CAL_WAVES * WAVE) void k_setup_cal(
    EventGeom g, const EventConst* __restrict__ ec, const BandHead* __restrict__ bh, double slope, int64_t M, int most,
    CalShape sh, const double* __restrict__ theta, int P, int ncal, int64_t B, int64_t Bp, double* __restrict__ coef,
    double* __restrict__ calc, int* __restrict__ plan, const int* __restrict__ perm) {
  alignas(16) __shared__ double rows_s[NCOEF * WAVE];
  __shared__ int ok_s[2][WAVE];
  __shared__ double diff_s[2][WAVE];
  __shared__ BandLds bands_s;
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / WAVE));
  const int lane = (int)(threadIdx.x % WAVE);
  const int64_t p = (int64_t)blockIdx.x * WAVE + lane;   // < Bp: Bp is a multiple of 64
  int64_t pc = p < B ? p : B - 1;                        // padding lanes repeat the last point
  if (perm) pc = perm[pc];
  BandPre pre;
  if (bh) pre = band_fetch(bh, w, lane);
  double* slopes_s = rows_s + CO_CR * WAVE;              // (these rows go to memory only)
  if (w < 2) {
    setup_halves<ND>(w, lane, theta + pc * P, g, ec, rows_s);
  } else {                                             // meanwhile the node values, half each
    if (bh) band_load(bh, slopes_s, 2 * WAVE);
    const int half = (ncal + 1) / 2, j0 = (w - 2) * half, j1 = w == 2 ? half : ncal;
    bool ok = true;
    double diff = 0.0, last = j0 > 0 ? theta[pc * P + NPARAM + j0 - 1] : 0.0;
    for (int j = j0; j < j1; ++j) {
      const double v = theta[pc * P + NPARAM + j];
      ok &= isfinite(v);
      calc[(int64_t)j * Bp + p] = v;
      // node j of a detector's amplitudes (the first nnode) or phases
      const int node = j % (2 * sh.nnode);
      if (node > sh.nnode) diff = fmax(diff, fabs(v - last));
      last = v;
    }
    ok_s[w - 2][lane] = ok ? 1 : 0;
    diff_s[w - 2][lane] = diff;
  }
  __syncthreads();
  const bool ok = ok_s[0][lane] && ok_s[1][lane];
  if (w < 2) setup_rows_write<ND>(w, lane, rows_s, ec, ok, coef, Bp, p);
  if (!bh) return;
  double a[NBASIS], T[ND];
#pragma unroll
  for (int m = 0; m < NBASIS; ++m) a[m] = rows_s[(CO_A + m) * WAVE + lane];
#pragma unroll
  for (int d = 0; d < ND; ++d) T[d] = rows_s[(CO_T + d) * WAVE + lane];
  if (!ok || !rows_in_range<ND>(a, T, ec)) a[0] = __builtin_nan("");
  band_ranges<ND>(slopes_s, pre.nbrk, a, T, w, SETUP_CAL_WAVES, lane, bands_s,
                  slope * fmax(diff_s[0][lane], diff_s[1][lane]));
  __syncthreads();
  band_hold(bh, pre, slopes_s, w, SETUP_CAL_WAVES, lane, bands_s);
  __syncthreads();
  if (w != 0) return;
  band_plan_cal(pre, slopes_s, M, most, sh.nchunk, lane, bands_s);
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // LDS from the lanes that wrote it
  plan[(int64_t)blockIdx.x * PLAN_INTS + lane] = bands_s.plan[lane];
}

// One bin of the calibrated loop. T_ is float (mixed: hardware phasors, float32 products) or
// double (float64: table phasor).
// 1 + dA and dphi come from their cubics in the bin's position t in the node interval (kA, kP:
// coefficients of t^0 .. t^3 for this chunk's interval, 1 included in kA[.][0]); the window
// weights cw (the same cubics' parts per node) serve only the adjoint's node moments.
template <int ND, bool GRAD, class T_, class Row, class CalRow, class GradP>
__device__ __forceinline__ void cal_bin(const Row r, const CalRow cw, T_ t, GradP gt, int k,
                                        const double (&a)[NBASIS], const double (&T)[ND], const T_ (&cr)[ND],
                                        const T_ (&ci)[ND], const T_ (&kA)[ND][4], const T_ (&kP)[ND][4],
                                        const double2* tbl, T_ (&z)[nz_cal(ND, GRAD)]) {
  constexpr bool MIXED = sizeof(T_) == 4;
  constexpr int MA = 3 * ND + NBASIS, MB = MA + 4 * ND;
  const double psi = phase_poly(a, r.x, r.w, r.w2, r.lnf);
  T_ y = 0, fk = 0;
  T_ gm[NBASIS];
  if constexpr (GRAD) {
    if constexpr (MIXED) {
      const RowGradF32 g = load_grad_f32(gt, k);
#pragma unroll
      for (int m = 0; m < NBASIS; ++m) gm[m] = g.g[m];
      fk = g.f;
    } else {
      const RowGradF64 g = load_grad_f64(gt, k);
      gm[0] = r.w; gm[1] = r.w2; gm[2] = g.g2; gm[3] = g.g3; gm[4] = r.lnf; gm[5] = r.x; gm[6] = g.g6; gm[7] = g.g7;
      fk = r.f;
    }
  }
#pragma unroll
  for (int d = 0; d < ND; ++d) {
    // g1 = 1 + dA and dphi at this bin (Horner in t)
    const T_ g1 = fma(fma(fma(kA[d][3], t, kA[d][2]), t, kA[d][1]), t, kA[d][0]);
    const T_ dp = fma(fma(fma(kP[d][3], t, kP[d][2]), t, kP[d][1]), t, kP[d][0]);
    // q = u p exp(i dphi) = u exp(-2 pi i (phi - dphi / 2 pi)): the calibration phase joins the
    // model phase before the phasor, so one phasor (with its gain correction) serves both. The
    // mixed variant subtracts dphi / 2 pi (at most a few hundredths of a cycle) in float32 from
    // the reduced phase; the float64 variant adds it in table units before the reduction.
    T_ cs, sn;
    if constexpr (MIXED) {
      const float rr = fmaf(dp, -0.15915494f, (float)__builtin_amdgcn_fract(fma(r.f, T[d], psi)));
      cs = __builtin_amdgcn_cosf(rr);
      sn = __builtin_amdgcn_sinf(rr);
    } else {
      sincos_tbl(fma(dp, -0.15915494309189535 * PH_TBL, fma(r.f, T[d], psi)), tbl, sn, cs);
    }
    const T_ ur = r.u[2 * d], ui = r.u[2 * d + 1];
    const T_ qr = fma(ur, cs, ui * sn);
    const T_ qi = fma(ui, cs, -(ur * sn));
    if constexpr (!GRAD) {
      z[2 * d] = fma(g1, qr, z[2 * d]);            // calibrated product g1 q
      z[2 * d + 1] = fma(g1, qi, z[2 * d + 1]);
    } else {
      const T_ vr = g1 * qr, vi = g1 * qi;          // calibrated product
      z[2 * d] += vr;
      z[2 * d + 1] += vi;
      const T_ yd = fma(cr[d], vi, ci[d] * vr);     // Im(c w_cal)
      const T_ ya = fma(cr[d], qr, -(ci[d] * qi));  // Re(c q)
      z[2 * ND + d] = fma(fk, yd, z[2 * ND + d]);
      y = d == 0 ? yd : y + yd;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        z[MA + 4 * d + i] = fma(cw.w[i], ya, z[MA + 4 * d + i]);
        z[MB + 4 * d + i] = fma(cw.w[i], yd, z[MB + 4 * d + i]);
      }
    }
  }
  if constexpr (GRAD) {
#pragma unroll
    for (int m = 0; m < NBASIS; ++m) z[3 * ND + m] = fma(gm[m], y, z[3 * ND + m]);
  }
}

// Where a group's rows lie: per node interval its first row and rows, from the group's plan or the
// grid's bins, and the rows of a chunk. `rows64`: the plan's, walked in float64.
struct CalRows {
  const int* pl;
  const CalShape& sh;
  bool rows64;
  int chunk;
  __device__ __forceinline__ CalRows(const CalShape& shape, const int* __restrict__ plan, int pg)
      : pl(plan ? plan + (int64_t)pg * PLAN_INTS : nullptr), sh(shape) {
    rows64 = pl && pl[2] != 0;
    const int M = sh.k0[sh.nnode - 1];
    chunk = pl ? pl[3] : (M + sh.nchunk - 1) / sh.nchunk;
  }
  __device__ __forceinline__ int row0(int j) const { return rows64 ? pl[4 + 2 * j] : sh.k0[j]; }
  __device__ __forceinline__ int rows(int j) const { return rows64 ? pl[5 + 2 * j] : sh.k0[j + 1] - sh.k0[j]; }
};

// Workgroup -> four chunks of a point group, as the plain loop deals them to the dies.
__device__ __forceinline__ bool locate_cal(const CalShape& sh, int& c, int& pg) {
  const int bid = blockIdx.x;
  const int item = (bid % NXCD) * sh.gper + bid / NXCD;
  if (item >= sh.items) return false;
  pg = item / sh.nbc;
  c = (item - pg * sh.nbc) * WAVES_PER_BLOCK + __builtin_amdgcn_readfirstlane((int)(threadIdx.x / WAVE));
  return true;
}

// Wavefronts per SIMD the register budget must allow: two for the mixed adjoint (three spilled 93
// registers, most of them inside the loop over intervals), otherwise no bound.
template <int ND, bool MIXED, bool GRAD>
constexpr int cal_waves_per_eu() {
  return (MIXED && GRAD) ? 2 : 1;
}

// The loop, a wavefront per chunk: equal shares of a group's rows, each walked interval by interval. Bound by
// float64 issue. Three detectors, 8 s, 10 nodes: values of 16,384 points 847 us a call on every bin, 158 on
// rows, 138 with the points in order (the loop 148 and 113); gradients of 8,192 822, 190 and 168 (119 and
// 91). Chunks that ended at the intervals' ends made uneven work: 342 us and 510.
// With a plan the float64 kernel takes the groups on float64 rows (all of them in a float64 call) and the
// mixed kernel the others: two launches, so that each keeps its own registers.
template <int ND, bool MIXED, bool GRAD>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(cal_waves_per_eu<ND, MIXED, GRAD>()))) void k_bins_cal(const void* __restrict__ tabv, const void* __restrict__ gtabv,
                                                    const void* __restrict__ calwv, const void* __restrict__ caltv,
                                                    const double* __restrict__ calB, const EventConst* __restrict__ ec,
                                                    const double* __restrict__ coef,
                                                    const double* __restrict__ calc, const int* __restrict__ plan,
                                                    int64_t B, int64_t Bp, CalShape sh, double* __restrict__ part) {
  typedef typename std::conditional<MIXED, float, double>::type T_;
  constexpr int NZ = nz_cal(ND, GRAD);
  __shared__ double2 tbl[MIXED ? 1 : PH_TBL];  // the float64 phasor table
  // mixed adjoint: the float64 totals of the 8 ND window moments stay in LDS (one column per
  // lane, so no barrier), which saves their registers
  constexpr int NNODE = GRAD ? 8 * ND : 0, NZU = NZ - NNODE;
  __shared__ double ntot[MIXED && GRAD ? 8 * ND : 1][MIXED && GRAD ? BLOCK : 1];
  int c, pg;
  if (!locate_cal(sh, c, pg)) return;                  // whole workgroup
  const CalRows cr_(sh, plan, pg);
  if (plan && cr_.rows64 == MIXED) return;             // whole workgroup: the other kernel's group
  if constexpr (!MIXED) {
    fill_phasor_table(tbl);
    __syncthreads();
  }
  if (c >= sh.nchunk) return;
  const int64_t p = (int64_t)pg * WAVE + (threadIdx.x % WAVE);
  const int64_t pc = p < B ? p : B - 1;
  double a[NBASIS], T[ND];
  T_ cr[ND], ci[ND];
  if constexpr (MIXED) {
    double crd[ND], cid[ND];
    load_coef<ND, double>(coef, Bp, pc, GRAD, a, T, crd, cid);
    mixed_factors<ND>(ec, crd, cid, cr, ci);
  } else {
    load_coef<ND, double>(coef, Bp, pc, GRAD, a, T, cr, ci);
    to_table_units<ND>(a, T);                          // the float64 phase runs in 1/PH_TBL cycles
  }
  double tot[NZ];
#pragma unroll
  for (int zz = 0; zz < NZ; ++zz) tot[zz] = 0.0;
  if constexpr (MIXED && GRAD) {
#pragma unroll
    for (int i = 0; i < NNODE; ++i) ntot[i][threadIdx.x] = 0.0;
  }
  // a float32 block's sums into the float64 totals
  auto flush = [&](const float (&z)[NZ]) {
    if constexpr (MIXED && GRAD) {
#pragma unroll
      for (int zz = 0; zz < NZU; ++zz) tot[zz] += (double)z[zz];
#pragma unroll
      for (int i = 0; i < NNODE; ++i) ntot[i][threadIdx.x] += (double)z[NZU + i];
    } else {
#pragma unroll
      for (int zz = 0; zz < NZ; ++zz) tot[zz] += (double)z[zz];
    }
  };
  const int n = sh.nnode;
  const double unit = MIXED ? ec->uref : 1.0;          // the float32 tables hold u / uref
  double* win = part + (int64_t)sh.nchunk * NZU * Bp;  // window moments [nchunk + n - 2][NNODE][Bp]
  // this chunk's rows, interval by interval
  const int q0 = c * cr_.chunk, q1 = q0 + cr_.chunk;
  int base = 0;
  for (int j = 0; j < n - 1 && base < q1; ++j) {
    const int row0 = cr_.row0(j), rows = cr_.rows(j);
    const int lo = q0 > base ? q0 - base : 0, hi = q1 - base < rows ? q1 - base : rows;
    base += rows;
    if (lo >= hi) continue;
    const int k0 = row0 + lo, k1 = row0 + hi;
    // this point's amplitude and phase node values in the interval's window, turned into the
    // cubics' coefficients: k[p] = sum_i v_i B[i][p] (1 added to the amplitude's k[0])
    T_ kA[ND][4], kP[ND][4];
    {
      const int j0 = sh.j0[j];
      const double* Bj = calB + (int64_t)j * 16;
#pragma unroll
      for (int d = 0; d < ND; ++d) {
        T_ va[4], vp[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          va[i] = (T_)calc[(int64_t)(2 * n * d + j0 + i) * Bp + pc];
          vp[i] = (T_)calc[(int64_t)(2 * n * d + n + j0 + i) * Bp + pc];
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          T_ sa = q == 0 ? (T_)1 : (T_)0, sp = 0;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            sa = fma(va[i], (T_)Bj[i * 4 + q], sa);
            sp = fma(vp[i], (T_)Bj[i * 4 + q], sp);
          }
          kA[d][q] = sa;
          kP[d][q] = sp;
        }
      }
    }
    if constexpr (MIXED) {
      const RowMixed<ND>* tab = (const RowMixed<ND>*)tabv;
      const RowGradF32* gt = (const RowGradF32*)gtabv;
      const RowCal32* cw = (const RowCal32*)calwv;
      const float* ct = (const float*)caltv;
      // float32 blocks of NB bins added into float64; each bin's rows are requested one bin ahead
      // (the tables carry zero padding rows past the last bin). Only the adjoint reads the weights.
      int k = k0;
      RowMixed<ND> cur = load_row_mixed<ND>(tab, k);
      RowCal32 cwc;
      if constexpr (GRAD) cwc = cw[k];
      float tc = ct[k];
      for (; k + NB <= k1; k += NB) {
        float z[NZ];
#pragma unroll
        for (int zz = 0; zz < NZ; ++zz) z[zz] = 0.0f;
#pragma unroll 2
        for (int jj = 0; jj < NB; ++jj) {
          const RowMixed<ND> nxt = load_row_mixed<ND>(tab, k + jj + 1);
          RowCal32 cwn;
          if constexpr (GRAD) cwn = cw[k + jj + 1];
          const float tn = ct[k + jj + 1];
          cal_bin<ND, GRAD, float>(cur, cwc, tc, gt, k + jj, a, T, cr, ci, kA, kP, tbl, z);
          cur = nxt;
          if constexpr (GRAD) cwc = cwn;
          tc = tn;
        }
        flush(z);
      }
      if (k < k1) {
        float z[NZ];
#pragma unroll
        for (int zz = 0; zz < NZ; ++zz) z[zz] = 0.0f;
        for (; k < k1; ++k)
          cal_bin<ND, GRAD, float>(load_row_mixed<ND>(tab, k), cw[k], ct[k], gt, k, a, T, cr, ci, kA, kP, tbl, z);
        flush(z);
      }
    } else {
      const RowF64<ND>* tab = (const RowF64<ND>*)tabv;
      const RowGradF64* gt = (const RowGradF64*)gtabv;
      const RowCal64* cw = (const RowCal64*)calwv;
      const double* ct = (const double*)caltv;
      RowF64<ND> cur = load_row_f64<ND>(tab, k0);
      RowCal64 cwc;
      if constexpr (GRAD) cwc = cw[k0];
      double tc = ct[k0];
      for (int k = k0; k < k1; ++k) {
        const RowF64<ND> nxt = load_row_f64<ND>(tab, k + 1);
        RowCal64 cwn;
        if constexpr (GRAD) cwn = cw[k + 1];
        const double tn = ct[k + 1];
        cal_bin<ND, GRAD, double>(cur, cwc, tc, gt, k, a, T, cr, ci, kA, kP, tbl, tot);
        cur = nxt;
        if constexpr (GRAD) cwc = cwn;
        tc = tn;
      }
    }
    if constexpr (GRAD) {                              // the interval's window moments
#pragma unroll
      for (int i = 0; i < NNODE; ++i) {
        double v;
        if constexpr (MIXED) {
          v = ntot[i][threadIdx.x];
          ntot[i][threadIdx.x] = 0.0;
        } else {
          v = tot[NZU + i];
          tot[NZU + i] = 0.0;
        }
        win[((int64_t)(c + j) * NNODE + i) * Bp + p] = unit * v;
      }
    }
  }
  if constexpr (MIXED) {   // the float64 loop's units (as mixed_units)
    const double gr = ec->gain_r, gi = ec->gain_i;
#pragma unroll
    for (int z = 0; z < 2 * ND; z += 2) {
      const double re = tot[z], im = tot[z + 1];
      tot[z] = unit * fma(re, gr, -(im * gi));
      tot[z + 1] = unit * fma(re, gi, im * gr);
    }
#pragma unroll
    for (int z = 2 * ND; z < NZU; ++z) tot[z] *= unit;
  }
#pragma unroll
  for (int zz = 0; zz < NZU; ++zz) part[((int64_t)c * NZU + zz) * Bp + p] = tot[zz];
}

// Epilogue, one workgroup of four wavefronts (eight for the adjoint) per 64 points, which share the gather. For the value the
// wavefronts also share the detectors' K_det terms, and the first forms it from the set-up rows. The
// adjoint's window moments are gathered one detector and kind (amplitude or phase) at a time, each
// summed in chunk order. Chunks come in interval order and an interval's window of four nodes
// starts at clamp(j - 1, 0, n - 4), which never moves back and moves by at most one node, so a
// node's moment is final once the window has moved past it: the task keeps the window in four
// registers and turns each finished node into its gradient at once. These tasks go to six of the
// wavefronts while the other two take the halves of the point model for the signal parameters.
constexpr int epc_waves(bool grad) { return grad ? 8 : 4; }

// With alpha the point's amplitude node values for a detector (loaded once, into registers):
// r_i = K1_i + (K2 alpha)_i. The effective K_det = K_det + 2 alpha.K1 + alpha.K2.alpha
// = K_det + sum_i alpha_i (K1_i + r_i), and the amplitude node gradient takes 2 r_i.
__device__ __forceinline__ void cal_alpha(const double* __restrict__ calc, int64_t Bp, int n, double (&al)[MAXNODE]) {
#pragma unroll
  for (int l = 0; l < MAXNODE; ++l) al[l] = l < n ? calc[(int64_t)l * Bp] : 0.0;
}
__device__ __forceinline__ double cal_r(const double* __restrict__ K1, const double* __restrict__ K2,
                                        const double (&al)[MAXNODE], int n, int i) {
  double r = K1[i];
#pragma unroll
  for (int l = 0; l < MAXNODE; ++l)
    if (l < n) r = fma(K2[i * n + l], al[l], r);
  return r;
}

template <int ND, bool GRAD>
__global__ __launch_bounds__(epc_waves(GRAD) * WAVE) void k_epilogue_cal(
    EventGeom g, const EventConst* __restrict__ ec, const double* __restrict__ kcal, const double* __restrict__ theta,
    int P, int64_t B, int64_t Bp, CalShape sh, const int* __restrict__ plan, const int* __restrict__ perm,
    const double* __restrict__ coef,
    const double* __restrict__ calc, const double* __restrict__ part, double* __restrict__ logl,
    double* __restrict__ grad) {
  constexpr int NZU = nz_of(ND, GRAD), NNODE = 8 * ND, NW = epc_waves(GRAD);
  __shared__ double acc_s[NZU][WAVE];
  __shared__ double ks_s[ND][WAVE];   // K_det's calibration term per point
  __shared__ double xs[GRAD ? GRAD_LDS : 1][WAVE];
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / WAVE));
  const int lane = (int)(threadIdx.x % WAVE);
  const int64_t p = (int64_t)blockIdx.x * WAVE + lane;   // p < Bp: the partial sums and set-up rows have Bp rows
  int64_t pt = p < B ? p : B - 1;                        // the point's row of theta and of the results
  if (perm) pt = perm[pt];
  const int n = sh.nnode, nchunk = sh.nchunk;
  gather_share<NZU, NW>(part, nchunk, Bp, p, w, lane, acc_s);
  if constexpr (GRAD) {
    double th[NPARAM];
    GradParts<ND> r;
    __syncthreads();
    if (w < 2) {
#pragma unroll
      for (int i = 0; i < NPARAM; ++i) th[i] = theta[pt * P + i];
      gradient_parts<ND>(w, lane, acc_s, th, g, xs, r);
    }
    const double amp = coef[CO_AMP * Bp + p];            // NaN for an invalid point
    // node gradients: amplitude A m_i - 1/2 A^2 |Q_det|^2 2 r_i, phase -A m_i
    const CalRows cr_(sh, plan, (int)blockIdx.x);
    const double* win = part + (int64_t)nchunk * NZU * Bp;
    for (int i = w - 2; w >= 2 && i < 2 * ND; i += NW - 2) {
      const int d = i >> 1, kind = i & 1;
      const double* alp = calc + (int64_t)(2 * n * d) * Bp + p;
      double al[MAXNODE];
      cal_alpha(alp, Bp, kind ? 0 : n, al);
      const double* K1 = kcal + (int64_t)d * (n + n * n);
      const double* K2 = K1 + n;
      const double qr = coef[(int64_t)(CO_QR + d) * Bp + p], qi = coef[(int64_t)(CO_QI + d) * Bp + p];
      const double hh = amp * amp * (qr * qr + qi * qi);
      double* out = grad + pt * P + NPARAM + 2 * n * d + (kind ? n : 0);
      const int wbase = (kind ? 4 * ND : 0) + 4 * d;
      double ks = 0.0;   // the amplitude task also sums K_det's calibration term
      auto finish = [&](int i, double m) {
        double x;
        if (kind) {
          x = -amp * m;
        } else {
          const double r = cal_r(K1, K2, al, n, i);
          ks = fma(alp[(int64_t)i * Bp], K1[i] + r, ks);
          x = amp * m - hh * r;
        }
        if (p < B) out[i] = x;
      };
      double mom[4] = {0.0, 0.0, 0.0, 0.0};
      int wb = 0;   // the window holds nodes wb .. wb + 3
      // the pieces (chunk, interval) in order, WB at a time so that their loads are in flight together
      constexpr int WB = 4;
      int j = 0, ch = 0, end = cr_.rows(0);             // next piece; end: rows up to the end of interval j
      while (j < n - 1) {
        int jj[WB], at[WB], m = 0;
#pragma unroll
        for (int q = 0; q < WB; ++q) {
          while (j < n - 1 && (end <= ch * cr_.chunk || cr_.rows(j) == 0)) {   // nothing of interval j from here on
            ++j;
            if (j < n - 1) end += cr_.rows(j);
          }
          jj[q] = j < n - 1 ? j : 0;
          at[q] = j < n - 1 ? ch + j : 0;
          m += j < n - 1 ? 1 : 0;
          if (j < n - 1 && end >= (ch + 1) * cr_.chunk) {
            ++ch;
          } else if (j < n - 1) {
            ++j;
            if (j < n - 1) end += cr_.rows(j);
          }
        }
        double v[WB][4];
#pragma unroll
        for (int q = 0; q < WB; ++q)
#pragma unroll
          for (int i = 0; i < 4; ++i) v[q][i] = q < m ? win[((int64_t)at[q] * NNODE + wbase + i) * Bp + p] : 0.0;
#pragma unroll
        for (int q = 0; q < WB; ++q) {
          if (q >= m) break;
          for (; wb < sh.j0[jj[q]]; ++wb) {
            finish(wb, mom[0]);
            mom[0] = mom[1];
            mom[1] = mom[2];
            mom[2] = mom[3];
            mom[3] = 0.0;
          }
#pragma unroll
          for (int i = 0; i < 4; ++i) mom[i] += v[q][i];
        }
      }
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (wb + i < n) finish(wb + i, mom[i]);
      for (int i = wb + 4; i < n; ++i) finish(i, 0.0);
      if (!kind) ks_s[d][lane] = ks;
    }
    __syncthreads();
    if (w > 1 || p >= B) return;
    double K[ND];
#pragma unroll
    for (int d = 0; d < ND; ++d) K[d] = ec->K[d] + ks_s[d][lane];
    gradient_finish<ND>(w, lane, th, K, xs, r, logl + pt, grad + pt * P);
  } else {
    // the K_det terms start with the wavefront after the one that took the last sum
    int t = w - NZU % NW;
    if (t < 0) t += NW;
    for (; t < ND; t += NW) {
      const double* alp = calc + (int64_t)(2 * n * t) * Bp + p;
      double al[MAXNODE];
      cal_alpha(alp, Bp, n, al);
      const double* K1 = kcal + (int64_t)t * (n + n * n);
      double ks = 0.0;
      for (int i = 0; i < n; ++i) ks = fma(alp[(int64_t)i * Bp], K1[i] + cal_r(K1, K1 + n, al, n, i), ks);
      ks_s[t][lane] = ks;
    }
    __syncthreads();
    if (w != 0 || p >= B) return;
    EventConst ek = *ec;
#pragma unroll
    for (int d = 0; d < ND; ++d) ek.K[d] += ks_s[d][lane];
    double acc[NZU];
#pragma unroll
    for (int z = 0; z < NZU; ++z) acc[z] = acc_s[z][lane];
    logl[pt] = epilogue_value_rows<ND, NZU>(acc, coef, Bp, p, ek, 1.0);
  }
}

template <int ND>
static hipError_t cal_nd(bool mixed, bool grad, const EventGeom& g, const EventConst* ec, const CalTables& t,
                         const double* theta, int P, int64_t B, int64_t Bp, int64_t M, const CalShape& sh, double* coef,
                         double* calc, double* part, int* plan, const int* perm, double* logl, double* gradout,
                         hipStream_t s) {
  const int ncal = 2 * sh.nnode * ND;
  if (Bp % WAVE != 0 || B < 1 || B > Bp || (t.bands && !plan)) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_setup_cal<ND>, dim3((unsigned)(Bp / WAVE)), dim3(SETUP_CAL_WAVES * WAVE), 0, s, g, ec, t.bands, t.slope,
                     M, float64_most(mixed, grad, true, M), sh, theta, P, ncal, B, Bp, coef, calc, plan, perm);
  const int* pl = t.bands ? plan : nullptr;
  const dim3 grid((unsigned)(sh.gper * NXCD)), block(BLOCK);
#define GWL_CB(MX, GR)                                                                                              \
  hipLaunchKernelGGL((k_bins_cal<ND, MX, GR>), grid, block, 0, s, MX ? t.tab32 : t.tab64,                           \
                     MX ? (const void*)t.g32 : (const void*)t.g64, MX ? (const void*)t.w32 : (const void*)t.w64,    \
                     MX ? (const void*)t.t32 : (const void*)t.t64, t.basis, ec, (const double*)coef,                \
                     (const double*)calc, pl, B, Bp, sh, part)
  if (mixed) {
    if (grad) GWL_CB(true, true); else GWL_CB(true, false);
  }
  if (!mixed || pl) {
    if (grad) GWL_CB(false, true); else GWL_CB(false, false);
  }
#undef GWL_CB
  const dim3 egrid((unsigned)((B + WAVE - 1) / WAVE)), eblock(epc_waves(grad) * WAVE);
#define GWL_CE(GR)                                                                                                   \
  hipLaunchKernelGGL((k_epilogue_cal<ND, GR>), egrid, eblock, 0, s, g, ec, t.kcal, theta, P, B, Bp, sh, pl, perm,    \
                     (const double*)coef, (const double*)calc, (const double*)part, logl, gradout)
  if (grad) GWL_CE(true); else GWL_CE(false);
#undef GWL_CE
  return hipGetLastError();
}

hipError_t launch_cal(int nd, bool mixed, bool grad, const EventGeom& g, const EventConst* ec, const CalTables& t,
                      const double* theta, int P, int64_t B, int64_t Bp, int64_t M, const CalShape& sh, double* coef,
                      double* calc, double* part, int* plan, const int* perm, double* logl, double* gradout,
                      hipStream_t s) {
  switch (nd) {
#define GWL_CN(N) \
  case N: return cal_nd<N>(mixed, grad, g, ec, t, theta, P, B, Bp, M, sh, coef, calc, part, plan, perm, logl, gradout, s);
    GWL_CN(1)
    GWL_CN(2)
    GWL_CN(3)
    GWL_CN(4)
#undef GWL_CN
  }
  return hipErrorInvalidValue;
}

}  // namespace gwl
