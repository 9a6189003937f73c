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

// A workgroup's NW wavefronts add the partial sums of 64 points over n chunks (in chunk order)
// into acc_s, wavefront w the sums w, w + NW, .... All of a wavefront's sums of four chunks are
// loaded before they are added: with one sum at a time a group of a few chunks waited for memory
// once per sum.
template <int NZ, int NW>
__device__ inline void gather_share(const double* __restrict__ part, int n, int64_t Bp, int64_t p, int w, int lane,
                                    double (*acc_s)[WAVE]) {
  constexpr int NS = (NZ + NW - 1) / NW, UC = 4;
  double a[NS];
#pragma unroll
  for (int i = 0; i < NS; ++i) a[i] = 0.0;
  for (int c0 = 0; c0 < n; c0 += UC) {
    double v[UC][NS];
#pragma unroll
    for (int u = 0; u < UC; ++u) {
      const int c = c0 + u < n ? c0 + u : n - 1;
#pragma unroll
      for (int i = 0; i < NS; ++i) {
        const int z = w + i * NW < NZ ? w + i * NW : NZ - 1;
        v[u][i] = part[((int64_t)c * NZ + z) * Bp + p];
      }
    }
#pragma unroll
    for (int u = 0; u < UC; ++u) {
      if (c0 + u >= n) break;
#pragma unroll
      for (int i = 0; i < NS; ++i) a[i] += v[u][i];
    }
  }
#pragma unroll
  for (int i = 0; i < NS; ++i)
    if (w + i * NW < NZ) acc_s[w + i * NW][lane] = a[i];
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
//   dlogL = sum_det [ Re(d(A E Q_det) Z_det) - 1/2 d(A^2 |Q|^2) K_det ]
//         + 2 pi A [ sum_m da_m Y_m + sum_det dT_det Z1_det ]
// (the second line is Re(-2 pi i A E G Q_det sum_k (da.g + f_k dT_det) w_det) written with c_det =
// E G Q_det). A, E and a_m depend on the intrinsic parameters only, Q_det and T_det on the extrinsic
// ones, and distance, phase and time enter in closed form, so two wavefronts share a group of 64
// points: each pushes four directions at once (dual numbers of four derivatives: the powers, logarithms
// and sines of the point model are evaluated once for them) through its half of the model and
// contracts them with its share of the sums; they then swap A, E and sum_det Q_det Z_det through
// LDS. (One parameter a pass through the whole model, eleven passes dealt to four wavefronts: 20.1 us
// for 16,384 points on three detectors against 8.0.)
constexpr int GRAD_LDS = 7 + MAXDET;    // doubles per point: A, Re E, Im E, validity, Re V, Im V, logL part, |Q_det|^2
template <int ND>
struct GradParts {
  double p[4][2];     // wavefront 0: dA, dc0 per direction; wavefront 1: sum_det dQ_det Z_det
  double u[4];        // wavefront 0: sum_m da_m Y_m; wavefront 1: sum_det dT_det Z1_det
  double rho[4][ND];  // wavefront 1: Re(conj(Q_det) dQ_det)
  double t;           // wavefront 1: sum_det Z1_det
};

// Wavefronts 0 and 1, before a barrier. acc_s: the sums [nz_of][WAVE] (Z, Z1, Y); xs: [GRAD_LDS][WAVE].
template <int ND>
__device__ inline void gradient_parts(int w, int lane, const double (*acc_s)[WAVE], const double (&th)[NPARAM],
                                      const EventGeom& g, double (*xs)[WAVE], GradParts<ND>& r) {
  typedef Dual<4> D;
  D t[NPARAM];
  PointModel<D> pm;
  // intrinsic directions: chirp mass, mass ratio, the spins; extrinsic: sky position, inclination,
  // polarisation
  if (w == 0) {
#pragma unroll
    for (int i = 0; i < NPARAM; ++i) t[i] = i < 4 ? dvar<4>(th[i], i) : dcst<4>(th[i]);
    point_intrinsic<D>(t, pm);
    const double c0 = pm.c0.v - rint(pm.c0.v);
    double es, ecs;
    sincos_cycles_f64(c0, es, ecs);
    xs[0][lane] = pm.amp.v;
    xs[1][lane] = ecs;
    xs[2][lane] = -es;
    xs[3][lane] = pm.valid ? 1.0 : 0.0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      r.p[i][0] = pm.amp.d[i];
      r.p[i][1] = pm.c0.d[i];
      double m = 0.0;
#pragma unroll
      for (int k = 0; k < NBASIS; ++k) m = fma(pm.a[k].d[i], acc_s[3 * ND + k][lane], m);
      r.u[i] = m;
    }
  } else if (w == 1) {
#pragma unroll
    for (int i = 0; i < NPARAM; ++i) t[i] = i >= 5 && i < 9 ? dvar<4>(th[i], i - 5) : dcst<4>(th[i]);
    point_extrinsic<D, ND>(t, g, pm);
    double vr = 0.0, vi = 0.0;
    r.t = 0.0;
#pragma unroll
    for (int i = 0; i < 4; ++i) r.p[i][0] = r.p[i][1] = r.u[i] = 0.0;
#pragma unroll
    for (int d = 0; d < ND; ++d) {
      const double zr = acc_s[2 * d][lane], zi = acc_s[2 * d + 1][lane], z1 = acc_s[2 * ND + d][lane];
      const double qr = pm.qr[d].v, qi = pm.qi[d].v;
      vr += fma(qr, zr, -(qi * zi));
      vi += fma(qr, zi, qi * zr);
      xs[7 + d][lane] = fma(qr, qr, qi * qi);
      r.t += z1;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const double dr = pm.qr[d].d[i], di = pm.qi[d].d[i];
        r.p[i][0] += fma(dr, zr, -(di * zi));
        r.p[i][1] += fma(dr, zi, di * zr);
        r.rho[i][d] = fma(qr, dr, qi * di);
        r.u[i] = fma(pm.tdet[d].d[i], z1, r.u[i]);
      }
    }
    xs[4][lane] = vr;
    xs[5][lane] = vi;
  }
}

// The same wavefronts, after the barrier: the value and the gradient row of one point (NaN for a
// point outside the model's domain). K: the detectors' K_det for this point.
template <int ND>
__device__ inline void gradient_finish(int w, int lane, const double (&th)[NPARAM], const double (&K)[ND],
                                       const double (*xs)[WAVE], const GradParts<ND>& r, double* __restrict__ logl,
                                       double* __restrict__ grad) {
  const double A = xs[0][lane], er = xs[1][lane], ei = xs[2][lane];
  const bool valid = xs[3][lane] != 0.0;
  const double nan = __builtin_nan("");
  auto put = [&](int i, double x) { grad[i] = valid ? x : nan; };
  if (w == 0) {
    const double vr = xs[4][lane], vi = xs[5][lane];
    const double sr = fma(er, vr, -(ei * vi)), si = fma(er, vi, ei * vr);   // sum_det E Q_det Z_det
    double h = 0.0;
#pragma unroll
    for (int d = 0; d < ND; ++d) h = fma(xs[7 + d][lane], K[d], h);
    const double da = fma(-A, h, sr);
    *logl = valid ? fma(A, sr, -0.5 * A * A * h) : nan;
#pragma unroll
    for (int i = 0; i < 4; ++i) put(i, fma(r.p[i][0], da, kTwoPi * A * fma(r.p[i][1], si, r.u[i])));
    put(4, -(A * da) / th[4]);
    put(9, -A * si);
  } else if (w == 1) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      double k = 0.0;
#pragma unroll
      for (int d = 0; d < ND; ++d) k = fma(r.rho[i][d], K[d], k);
      const double pr = fma(er, r.p[i][0], -(ei * r.p[i][1]));
      put(5 + i, A * (pr - A * k + kTwoPi * r.u[i]));
    }
    put(10, kTwoPi * A * r.t);
  }
}

}  // namespace gwl
