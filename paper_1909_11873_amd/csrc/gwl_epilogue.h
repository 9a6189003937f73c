// Float64 per-point work shared by the single-event and multi-event kernels: the set-up rows
// before the bin loop, and the epilogue after it (the log-likelihood ratio from the
// accumulated sums and, for the adjoint, its gradient with respect to all 11 parameters).
#pragma once

#include <hip/hip_runtime.h>

#include "gwl_common.h"
#include "gwl_device.h"

namespace gwl {

// The constant phase factor E = exp(-2 pi i c0) (c0 in cycles). adjoint_factor spells out its fused
// multiply-adds, so that every kernel forming c_det rounds the same way (the in-kernel set-up and
// the set-up kernel give bitwise equal gradients).
__device__ inline void phase_factor(double c0raw, double& er, double& ei) {
  const double c0 = c0raw - rint(c0raw);
  double es, ecs;
  sincos_cycles_f64(c0, es, ecs);
  er = ecs;
  ei = -es;
}
// c_det = E Q_det
__device__ inline void adjoint_factor(double egr, double egi, double qr, double qi, double& cr, double& ci) {
  cr = fma(egr, qr, -(egi * qi));
  ci = fma(egr, qi, egi * qr);
}

// Whether the phase sum_m a_m g_m(f) + f T_det stays below PHASE_LIMIT cycles on the event's
// grid (a and T after the fiducial's offsets; always true without an event).
template <int ND>
__device__ inline bool rows_in_range(const double* a, const double* T, const EventConst* ec) {
  if (!ec) return true;
  double bound = 0.0, tmax = 0.0;
#pragma unroll
  for (int m = 0; m < NBASIS; ++m) bound = fma(fabs(a[m]), ec->gmax[m], bound);
#pragma unroll
  for (int d = 0; d < ND; ++d) tmax = fmax(tmax, fabs(T[d]));
  return fma(tmax, ec->fmax, bound) < PHASE_LIMIT;
}

// The in-kernel set-up in two halves, each writing its rows of one point into the LDS rows
// [NCOEF][WAVE] (lane = point), so that two wavefronts can run them at once. The intrinsic half
// writes CO_A (less the fiducial's), CO_C0 and CO_AMP, NaN for a point outside the model's
// domain; the extrinsic half writes CO_T (less the fiducial's), CO_QR and CO_QI. The phase
// range check and the adjoint factors c_det then come from these rows (rows_in_range,
// phase_factor).
__device__ inline void setup_lds_intrinsic(const double (&th)[NPARAM], const EventConst* ec, double* rows_s, int lane) {
  PointModel<double> pm;
  point_intrinsic<double>(th, pm);
  const double nan = __builtin_nan("");
#pragma unroll
  for (int m = 0; m < NBASIS; ++m) rows_s[(CO_A + m) * WAVE + lane] = pm.valid ? pm.a[m] - (ec ? ec->fa[m] : 0.0) : nan;
  rows_s[CO_C0 * WAVE + lane] = pm.valid ? pm.c0 : nan;
  rows_s[CO_AMP * WAVE + lane] = pm.valid ? pm.amp : nan;
}
template <int ND>
__device__ inline void setup_lds_extrinsic(const double (&th)[NPARAM], const EventGeom& g, const EventConst* ec,
                                           double* rows_s, int lane) {
  PointModel<double> pm;
  point_extrinsic<double, ND>(th, g, pm);
#pragma unroll
  for (int d = 0; d < ND; ++d) {
    rows_s[(CO_T + d) * WAVE + lane] = pm.tdet[d] - (ec ? ec->fT[d] : 0.0);
    rows_s[(CO_QR + d) * WAVE + lane] = pm.qr[d];
    rows_s[(CO_QI + d) * WAVE + lane] = pm.qi[d];
  }
}

// Sum the per-chunk partials of one point in chunk order (deterministic). The chunk loop is
// unrolled so that several chunks' loads are in flight before their adds, which still run in
// chunk order; with one thread per point this loop is latency-bound otherwise.
template <int NZ>
__device__ inline void gather(const double* __restrict__ part, int nchunk, int64_t Bp, int64_t p, double (&acc)[NZ]) {
#pragma unroll
  for (int z = 0; z < NZ; ++z) acc[z] = 0.0;
#pragma unroll 8
  for (int c = 0; c < nchunk; ++c) {
#pragma unroll
    for (int z = 0; z < NZ; ++z) acc[z] += part[((int64_t)c * NZ + z) * Bp + p];
  }
}

// logL = sum_det [ uref Re(A E Q_det Z_det) - 1/2 A^2 |Q_det|^2 K_det ], E = exp(-2 pi i c0), with
// `acc` holding Z_det (re, im) first, from the point's set-up rows (A, Q_det and c0 as the point model gave them; a
// point outside the model's domain has NaN rows and gets NaN), so the forward epilogue does not
// evaluate the point model a second time.
template <int ND, int NZ>
__device__ inline double epilogue_value_rows(const double (&acc)[NZ], const double* __restrict__ coef, int64_t Bp,
                                             int64_t p, const EventConst& ec, double uref) {
  const double amp = coef[CO_AMP * Bp + p];
  const double c0f = coef[CO_C0 * Bp + p];
  const double c0 = c0f - rint(c0f);
  double es, ecs;
  sincos_cycles_f64(c0, es, ecs);
  const double er = ecs, ei = -es;
  double out = 0.0;
#pragma unroll
  for (int d = 0; d < ND; ++d) {
    const double qr = coef[(CO_QR + d) * Bp + p], qi = coef[(CO_QI + d) * Bp + p];
    const double xr = amp * (er * qr - ei * qi);
    const double xi = amp * (er * qi + ei * qr);
    const double dh = uref * (xr * acc[2 * d] - xi * acc[2 * d + 1]);
    const double hh = amp * amp * (qr * qr + qi * qi) * ec.K[d];
    out += dh - 0.5 * hh;
  }
  return out;
}

// Gradient. With w_det = u p, p = exp(-2 pi i (psi_k + f_k T_det)) and y_det = Im(c_det w_det),
// the bin loop accumulated per point
//   Z_det = sum_k w_det,  Z1_det = sum_k f_k y_det,  Y_m = sum_k g_m(f_k) sum_det y_det.
// The phase coefficients a_m and the shifts T_det enter logL only through p, so
//   dlogL = sum_det [ uref Re(d(A E Q_det) Z_det) - 1/2 d(A^2 |Q|^2) K_det ]
//         + 2 pi uref A [ sum_m da_m Y_m + sum_det dT_det Z1_det ]
// (the second line is Re(-2 pi i uref A E G Q_det sum_k (da.g + f_k dT_det) w_det) written
// with c_det = E G Q_det).
// Every d(.) comes from one-direction dual numbers pushed through the same point model, one
// parameter at a time (11 passes; this keeps the register footprint of the epilogue small).
// One pass: the derivative with respect to parameter j; `value` and `valid` are the same in every
// pass (the primal part does not depend on the direction).
template <int ND>
__device__ inline double epilogue_gradient_pass(const double (&acc)[nz_of(ND, true)], const double (&th)[NPARAM],
                                                const EventGeom& g, const EventConst& ec, double uref, int j,
                                                bool& valid, double& value) {
  typedef Dual<1> D;
  D t[NPARAM];
#pragma unroll
  for (int i = 0; i < NPARAM; ++i) {
    t[i].v = th[i];
    t[i].d[0] = (i == j) ? 1.0 : 0.0;
  }
  PointModel<D> pm;
  point_model<D, ND>(t, g, pm);
  D c0 = pm.c0;
  c0.v -= rint(c0.v);
  const D arg = c0 * kTwoPi;
  const D er = xcos(arg), ei = -xsin(arg);
  D tot = dcst<1>(0.0);
#pragma unroll
  for (int d = 0; d < ND; ++d) {
    const D xr = pm.amp * (er * pm.qr[d] - ei * pm.qi[d]);
    const D xi = pm.amp * (er * pm.qi[d] + ei * pm.qr[d]);
    const D dh = (xr * acc[2 * d] - xi * acc[2 * d + 1]) * uref;
    const D hh = pm.amp * pm.amp * (pm.qr[d] * pm.qr[d] + pm.qi[d] * pm.qi[d]) * ec.K[d];
    tot = tot + dh - 0.5 * hh;
  }
  double sm = 0.0;
#pragma unroll
  for (int m = 0; m < NBASIS; ++m) sm += pm.a[m].d[0] * acc[3 * ND + m];
#pragma unroll
  for (int d = 0; d < ND; ++d) sm += pm.tdet[d].d[0] * acc[2 * ND + d];
  value = tot.v;
  valid = pm.valid;
  return tot.d[0] + kTwoPi * uref * pm.amp.v * sm;
}

}  // namespace gwl
