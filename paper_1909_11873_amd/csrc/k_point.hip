// Per-point kernels: set-up (phase coefficients, time shifts, projection factors) before the
// evaluation kernel, and the adjoint's float64 epilogue after it (the log-likelihood ratio of
// Eq. 2 and its gradient with respect to all 11 parameters; the value alone is finished inside
// the evaluation kernel).
#include <hip/hip_runtime.h>

#include "gwl_bands.h"
#include "gwl_bins.h"
#include "gwl_common.h"
#include "gwl_device.h"
#include "gwl_epilogue.h"
#include "gwl_launch.h"
#include "gwl_setup.h"

namespace gwl {

// Set-up: one workgroup per 64 points. The intrinsic half of the point model (phase coefficients,
// constant phase, amplitude) runs on one wavefront and the extrinsic half (sky, orientation,
// per-detector delays and projection factors) on another, at once, into LDS rows; each of the two
// then writes half of the rows, with the phase-range check and the adjoint factors taken from
// the LDS rows (NaN rows for a point outside the model's domain or range). On an event with
// band-limited rows four wavefronts share the bounds of t(f) over the group, and the group's plan
// is left in plan[pg] (float32 units and gains are the evaluation kernel's affair). Bound by latency, about 10 us from
// theta to plan at any number of groups that are resident together: the model 4, the bounds 3, the
// choice 2.
constexpr int SETUP_WAVES = 2, SETUP_WAVES_BANDS = 4;

template <int ND>
__global__ __launch_bounds__(SETUP_WAVES_BANDS * WAVE) void k_setup(EventGeom g, const EventConst* __restrict__ ec,
                                                                    const BandHead* __restrict__ bh, int most, int nchunk,
                                                                    const double* __restrict__ theta, int64_t B,
                                                                    int64_t Bp, double* __restrict__ coef,
                                                                    int* __restrict__ plan,
                                                                    const int* __restrict__ perm) {
  alignas(16) __shared__ double rows_s[NCOEF * WAVE];
  __shared__ BandLds bands_s;
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / WAVE));
  const int lane = (int)(threadIdx.x % WAVE);
  const int64_t p = (int64_t)blockIdx.x * WAVE + lane;   // < Bp: Bp is a multiple of 64
  int64_t pc = p < B ? p : B - 1;                        // padding lanes repeat the last point
  if (perm) pc = perm[pc];
  BandPre pre;
  if (bh) pre = band_fetch(bh, w, lane);
  double* slopes_s = rows_s + CO_CR * WAVE;                // (these rows go to memory only)
  if (w < 2) setup_halves<ND>(w, lane, theta + pc * NPARAM, g, ec, rows_s);
  else if (bh) band_load(bh, slopes_s, 2 * WAVE);
  __syncthreads();
  if (w < 2) setup_rows_write<ND>(w, lane, rows_s, ec, true, coef, Bp, p);
  if (!bh) return;
  double a[NBASIS], T[ND];
#pragma unroll
  for (int m = 0; m < NBASIS; ++m) a[m] = rows_s[(CO_A + m) * WAVE + lane];
#pragma unroll
  for (int d = 0; d < ND; ++d) T[d] = rows_s[(CO_T + d) * WAVE + lane];
  if (!rows_in_range<ND>(a, T, ec)) a[0] = __builtin_nan("");
  band_ranges<ND>(slopes_s, pre.nbrk, a, T, w, SETUP_WAVES_BANDS, lane, bands_s);
  __syncthreads();
  band_hold(bh, pre, slopes_s, w, SETUP_WAVES_BANDS, lane, bands_s);
  __syncthreads();
  if (w != 0) return;
  band_plan(pre, slopes_s, most, nchunk, lane, bands_s);
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // LDS from the lanes that wrote it
  plan[(int64_t)blockIdx.x * PLAN_INTS + lane] = bands_s.plan[lane];
}

hipError_t launch_setup(int nd, const EventGeom& g, const EventConst* ec, const double* theta, int64_t B, int64_t Bp,
                        double* coef, hipStream_t s, const BandHead* bands, int most, int nchunk, int* plan, const int* perm) {
  if (Bp % WAVE != 0 || B < 1 || B > Bp) return hipErrorInvalidValue;
  if (bands && (!ec || !plan || nchunk < 1)) return hipErrorInvalidValue;
  dim3 grid((unsigned)(Bp / WAVE)), block((unsigned)((bands ? SETUP_WAVES_BANDS : SETUP_WAVES) * WAVE));
#define GWL_SETUP(N) \
  case N: hipLaunchKernelGGL(k_setup<N>, grid, block, 0, s, g, ec, bands, most, nchunk, theta, B, Bp, coef, plan, perm); break;
  switch (nd) {
    GWL_SETUP(1)
    GWL_SETUP(2)
    GWL_SETUP(3)
    GWL_SETUP(4)
    default: return hipErrorInvalidValue;
  }
#undef GWL_SETUP
  return hipGetLastError();
}

// With the ISCO cut-off (fgrid and kcum given), <h|h> takes the kept bins' share of K_det; the
// cut moves with the masses in steps, so it adds nothing to the derivative.
//
// One workgroup per 64 points: EPG_WAVES wavefronts first add the points' partial sums over the
// chunks (in chunk order, each wavefront its share of the sums) into LDS, then two of them take
// the halves of the point model.
constexpr int EPG_WAVES = 4;
template <int ND>
__global__ __launch_bounds__(EPG_WAVES * WAVE) void k_epilogue_grad(EventGeom g, const EventConst* __restrict__ ec,
                                                                    const double* __restrict__ theta, int64_t B,
                                                                    int64_t Bp, int nchunk,
                                                                    const double* __restrict__ part,
                                                                    double* __restrict__ logl,
                                                                    double* __restrict__ grad,
                                                                    const double* __restrict__ fgrid,
                                                                    const double* __restrict__ kcum, int64_t M,
                                                                    const int* __restrict__ perm) {
  constexpr int NZ = nz_of(ND, true);
  __shared__ double acc_s[NZ][WAVE];
  __shared__ double xs[GRAD_LDS][WAVE];
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / WAVE));
  const int lane = (int)(threadIdx.x % WAVE);
  const int64_t p = (int64_t)blockIdx.x * WAVE + lane;   // p < Bp: the partial sums have Bp rows
  int64_t pc = p < B ? p : B - 1;
  if (perm) pc = perm[pc];
  gather_share<NZ, EPG_WAVES>(part, nchunk, Bp, p, w, lane, acc_s);
  double th[NPARAM];
#pragma unroll
  for (int i = 0; i < NPARAM; ++i) th[i] = theta[pc * NPARAM + i];
  __syncthreads();
  GradParts<ND> r;
  gradient_parts<ND>(w, lane, acc_s, th, g, xs, r);
  __syncthreads();
  if (w > 1 || p >= B) return;
  double K[ND];
#pragma unroll
  for (int d = 0; d < ND; ++d) K[d] = ec->K[d];
  if (fgrid) {
    const int kc = isco_bins(th[0], th[1], fgrid, M, *ec);
#pragma unroll
    for (int d = 0; d < ND; ++d) K[d] = kcum[(int64_t)d * (M + 1) + kc];
  }
  gradient_finish<ND>(w, lane, th, K, xs, r, logl + pc, grad + pc * NPARAM);
}

// The points' order for a large batch (launch_order). A group's rows are as many as its earliest and latest
// t(f) need, and 64 points in the caller's order mostly span the whole prior: neighbours of about the
// same arrival time and mass need a third fewer (three detectors, 8 s: 1,587 rows a group without, 1,109
// with blocks of 1,024 points; whole blocks of 4,096 save another 4 %). One workgroup orders kOrderBlock points: by eighths
// of their range of arrival times, within an eighth by sixteenths of their range of masses, up and down
// in turn, within a sixteenth as they come; a point with a parameter that is not finite goes last. A
// counting sort: places within a wavefront's equals from ballots, the counts of 128 keys by 16
// wavefronts scanned in LDS. Bound by latency: 5.9 us at 65,536 points
// (a bitonic sort of whole keys: 8.1).
constexpr int kOrderBlock = 1024, kOrderWaves = kOrderBlock / WAVE, kOrderKeys = 128;
__global__ __launch_bounds__(kOrderBlock) void k_order(const double* __restrict__ theta, int P, int64_t B,
                                                       int* __restrict__ perm) {
  __shared__ float4 ext_s[kOrderWaves];
  __shared__ int cnt_s[kOrderKeys * kOrderWaves];      // per key, the wavefronts in turn
  __shared__ int sum_s[kOrderWaves];
  const int i = (int)threadIdx.x, w = i / WAVE, lane = i % WAVE;
  const int64_t p0 = (int64_t)blockIdx.x * kOrderBlock, p = p0 + i;
  const float inf = __builtin_inff();
  const float m = p < B ? (float)theta[p * P] : inf, t = p < B ? (float)theta[p * P + NPARAM - 1] : inf;
  cnt_s[2 * i] = cnt_s[2 * i + 1] = 0;
  const bool ok = isfinite(m) && isfinite(t);
  float m0 = wave_max_hi(ok ? -m : -inf), m1 = wave_max_hi(ok ? m : -inf);
  float t0 = wave_max_hi(ok ? -t : -inf), t1 = wave_max_hi(ok ? t : -inf);
  if (lane == WAVE - 1) ext_s[w] = make_float4(m0, m1, t0, t1);
  __syncthreads();
  m0 = m1 = t0 = t1 = -inf;
#pragma unroll
  for (int v = 0; v < kOrderWaves; ++v) {
    const float4 e = ext_s[v];
    m0 = fmaxf(m0, e.x);
    m1 = fmaxf(m1, e.y);
    t0 = fmaxf(t0, e.z);
    t1 = fmaxf(t1, e.w);
  }
  m0 = -m0;
  t0 = -t0;
  int key = kOrderKeys - 1;
  if (ok) {                                            // (a NaN, from ranges beyond float32, counts as 0)
    const float ft = t1 > t0 ? (t - t0) / (t1 - t0) : 0.0f, fm = m1 > m0 ? (m - m0) / (m1 - m0) : 0.0f;
    const int cell = (int)fminf(fmaxf(8.0f * ft, 0.0f), 7.0f), q = (int)fminf(fmaxf(16.0f * fm, 0.0f), 15.0f);
    key = cell * 16 + (cell & 1 ? 15 - q : q);
  }
  unsigned long long same = ~0ull;                     // the wavefront's lanes of this key
#pragma unroll
  for (int b = 1; b < kOrderKeys; b <<= 1) {
    const unsigned long long v = __ballot((key & b) != 0);
    same &= key & b ? v : ~v;
  }
  const int rank = __popcll(same & ((1ull << lane) - 1));
  if (rank == 0) cnt_s[key * kOrderWaves + w] = __popcll(same);
  __syncthreads();
  // exclusive sums over the counts, two a thread
  const int c0 = cnt_s[2 * i], c1 = cnt_s[2 * i + 1];
  int incl = c0 + c1;
#pragma unroll
  for (int off = 1; off < WAVE; off <<= 1) {
    const int o = __shfl_up(incl, off);
    if (lane >= off) incl += o;
  }
  if (lane == WAVE - 1) sum_s[w] = incl;
  __syncthreads();
  int before = incl - c0 - c1;
#pragma unroll
  for (int v = 0; v < kOrderWaves; ++v) before += v < w ? sum_s[v] : 0;
  cnt_s[2 * i] = before;
  cnt_s[2 * i + 1] = before + c0;
  __syncthreads();
  // places below the block's number of points belong to its points: the lanes past them come last
  if (p < B) perm[p0 + cnt_s[key * kOrderWaves + w] + rank] = (int)p;
}

hipError_t launch_order(const double* theta, int P, int64_t B, int* perm, hipStream_t s) {
  if (!theta || !perm || P < NPARAM || B < 1) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_order, dim3((unsigned)((B + kOrderBlock - 1) / kOrderBlock)), dim3(kOrderBlock), 0, s, theta, P, B,
                     perm);
  return hipGetLastError();
}

hipError_t launch_epilogue(int nd, bool grad, const EventGeom& g, const EventConst* ec, const double* theta,
                           const double*, int64_t B, int64_t Bp, int nchunk, const double* part, double* logl,
                           double* gradout, hipStream_t s, const double* fgrid, const double* kcum, int64_t M,
                           const int* perm) {
  if (!grad) return hipErrorInvalidValue;  // the value's epilogue runs in the evaluation kernel
  dim3 grid((unsigned)((B + WAVE - 1) / WAVE));
#define GWL_EPI(N)                                                                                                  \
  case N:                                                                                                           \
    hipLaunchKernelGGL(k_epilogue_grad<N>, grid, dim3(EPG_WAVES * WAVE), 0, s, g, ec, theta, B, Bp, nchunk, part, \
                       logl, gradout, fgrid, kcum, M, perm);                                                        \
    break;
  switch (nd) {
    GWL_EPI(1)
    GWL_EPI(2)
    GWL_EPI(3)
    GWL_EPI(4)
    default: return hipErrorInvalidValue;
  }
#undef GWL_EPI
  return hipGetLastError();
}

}  // namespace gwl
