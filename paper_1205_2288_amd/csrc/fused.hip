// Force, potential and time-step criterion of the active set in one pass over the pairs.
//
// A variant of Algorithm 2's order: the paper evaluates the criterion (Eq. nbdt) after the
// corrector (step 7 after step 6), with the corrected velocities of the active particles;
// here it is evaluated with the state the force sees, i.e. the predicted velocities
// v + a h of the active particles.  Positions are the same either way (the corrector sets
// r to the prediction), so the free-fall term is unchanged and the collision term differs
// only through (a_new - a) h / 2 in the active velocities, O(h^2) relative.  In exchange
// the pair's separation, loads and loop are shared by the two sums.
//
// Same scalar-load structure as k_force_scalar (one target per lane of the workgroup or, for
// fewer than kShareMaxAct targets, of every wave; j-particles through wave-uniform loads in
// units of CH, self / padding masked by a wave vote), in the force's split, with the force
// and criterion pair arithmetic of the two separate kernels, so that the force is bitwise
// the one tsbts_force returns.  Partials [S][6][n_act]: the force and potential sums, max
// v^2/r^2 and min s m^(-2/3).  Measured (us of device time, a target per lane of the
// workgroup, of every wave): mixed N = 4096 k = 100 14.2, 13.7, 2000 24.0, 15.1; 131072 100
// 55.8, 45.9, 777 155, 104; float64 N = 4096 100 16.8, 11.1; 131072 777 224, 162.
#include "cells.hpp"
#include "correct.hpp"
#include "criterion.hpp"
#include "force_pair.hpp"

namespace tsbts {
namespace {

struct FusedArgs {
  int64_t n, npad;
  const float *p32;
  const double *p64;
  const double *v64;
  const int32_t *idx;
  int n_act;
  SplitPlan plan;
  int n_units;    // j-units of CH particles, or of kShare * CH (share)
  int share;      // the waves of a workgroup share 64 targets (ShareShape)
  float eps2f;
  double eps2;
  double eta;
  double *part;  // [S][6][n_act]
  double *acc;   // [3][n_act]
  double *pot;   // [n_act] or null
  double *dtc;   // [n_act]
  int correct;   // apply the corrector in the reduction
  CorrectArgs corr;
};

template <class V, int NEWTON>
__device__ __forceinline__ void finish_all(const FusedArgs &A, int q, int64_t g, double sx,
                                           double sy, double sz, double sp, double qm,
                                           double sm) {
  const double k = Scale<V, NEWTON>::kAcc;
  const double an[3] = {k * sx, k * sy, k * sz};
  A.acc[q] = an[0];
  A.acc[A.n_act + q] = an[1];
  A.acc[2 * A.n_act + q] = an[2];
  if (A.pot) A.pot[q] = -sp;
  A.dtc[q] = finish_dt(A.eta, qm, sm);
  if (A.correct) correct_one(A.corr, q, g, an);
}

template <class V, int NEWTON, int MASK, int POT, int CH, class F>
__device__ __forceinline__ void fused_unit(const FusedArgs &A, const typename V::I &If,
                                           const typename StepRec<V>::I &Ic, int g,
                                           int64_t jbase, F eps2, F &fx, F &fy, F &fz, F &fp,
                                           F &qm, F &sm) {
#pragma unroll 4
  for (int jj = 0; jj < CH; ++jj) {
    const int64_t j = jbase + jj;
    const typename V::J Jf = V::load_j(A.p32, A.p64, A.npad, j, Scale<V, NEWTON>::kMass);
    const typename StepRec<V>::J Jc = load_jv<V>(A, j);
    const bool skip = MASK && (j == g || j >= A.n);
    pair_acc<V, NEWTON, MASK, POT>(If, Jf, eps2, skip, fx, fy, fz, fp);
    pair_step(Ic, Jc, eps2, skip, qm, sm);
  }
}

template <class V, int NEWTON, int POT, int CH, int SH>
__global__ __launch_bounds__(kWG) void k_fused(FusedArgs A) {
  using F = typename V::F;
  const int lane = static_cast<int>(threadIdx.x) & 63;
  const int w = SH == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int itile, slice;
  split_tile(blockIdx.x, A.plan, itile, slice);
  if (slice >= A.plan.n_slices) return;
  const int jt0 = slice * A.plan.tiles_per_slice;
  const int jt1 = min(jt0 + A.plan.tiles_per_slice, A.n_units);
  const F eps2 = sizeof(F) == 4 ? static_cast<F>(A.eps2f) : static_cast<F>(A.eps2);
  const int q = SH == 1 ? itile * kWG + static_cast<int>(threadIdx.x) : itile * 64 + lane;
  const int g = A.idx[min(q, A.n_act - 1)];
  const typename V::I If = V::load_i(A.p32, A.p64, A.npad, g);
  const typename StepRec<V>::I Ic = load_iv<V>(A, g);
  double sx = 0.0, sy = 0.0, sz = 0.0, sp = 0.0;
  F qm = F(0);
  F sm = sizeof(F) == 4 ? static_cast<F>(__builtin_inff()) : static_cast<F>(__builtin_inf());
  for (int jt = jt0; jt < jt1; ++jt) {
    const int64_t jbase = (static_cast<int64_t>(jt) * SH + w) * CH;
    if (SH > 1 && jbase >= A.npad) break;
    F fx = F(0), fy = F(0), fz = F(0), fp = F(0);
    if (__ballot(g >= jbase && g < jbase + CH) != 0 || jbase + CH > A.n)
      fused_unit<V, NEWTON, 1, POT, CH>(A, If, Ic, g, jbase, eps2, fx, fy, fz, fp, qm, sm);
    else
      fused_unit<V, NEWTON, 0, POT, CH>(A, If, Ic, g, jbase, eps2, fx, fy, fz, fp, qm, sm);
    sx += static_cast<double>(fx);
    sy += static_cast<double>(fy);
    sz += static_cast<double>(fz);
    sp += static_cast<double>(fp);
  }
  double *out = A.part + static_cast<int64_t>(slice) * 6 * A.n_act;
  if constexpr (SH > 1) {
    // wave c: sum c of the waves, in wave order; wave 0 the maxima too, wave 1 the minima
    static_assert(SH == 4, "a wave per sum");
    __shared__ double red[SH][6][64];
    red[w][0][lane] = sx;
    red[w][1][lane] = sy;
    red[w][2][lane] = sz;
    red[w][3][lane] = sp;
    red[w][4][lane] = static_cast<double>(qm);
    red[w][5][lane] = static_cast<double>(sm);
    __syncthreads();
    if (q >= A.n_act) return;
    double x = red[0][w][lane];
#pragma unroll
    for (int u = 1; u < SH; ++u) x += red[u][w][lane];
    out[w * static_cast<int64_t>(A.n_act) + q] = x;
    if (w >= 2) return;
    double y = red[0][4 + w][lane];
#pragma unroll
    for (int u = 1; u < SH; ++u) {
      const double z = red[u][4 + w][lane];
      y = w == 0 ? fmax(y, z) : fmin(y, z);
    }
    out[(4 + w) * static_cast<int64_t>(A.n_act) + q] = y;
    return;
  }
  if (q >= A.n_act) return;
  out[q] = sx;
  out[A.n_act + q] = sy;
  out[2 * A.n_act + q] = sz;
  out[3 * A.n_act + q] = sp;
  out[4 * A.n_act + q] = static_cast<double>(qm);
  out[5 * A.n_act + q] = static_cast<double>(sm);
}

// Combine the slices in slice order (sums; max and min are exact) and finish: one thread
// per target, one wave per target with the lanes striding over many slices, or (below)
// rows of 64 targets, in the force reduction's order for the same call.  Always a
// separate launch: the corrector it may apply rewrites velocity planes the pair loop reads.
template <class V, int NEWTON>
__global__ __launch_bounds__(kWG) void k_fused_reduce(FusedArgs A) {
  const int q = blockIdx.x * kWG + threadIdx.x;
  if (q >= A.n_act) return;
  double sx = 0.0, sy = 0.0, sz = 0.0, sp = 0.0, qm = 0.0, sm = __builtin_inf();
  const int64_t stride = 6 * static_cast<int64_t>(A.n_act);
  for (int s = 0; s < A.plan.n_slices; ++s) {
    const double *in = A.part + s * stride;
    sx += in[q];
    sy += in[A.n_act + q];
    sz += in[2 * A.n_act + q];
    sp += in[3 * A.n_act + q];
    qm = fmax(qm, in[4 * A.n_act + q]);
    sm = fmin(sm, in[5 * A.n_act + q]);
  }
  finish_all<V, NEWTON>(A, q, A.idx[q], sx, sy, sz, sp, qm, sm);
}

template <class V, int NEWTON>
__global__ __launch_bounds__(kWG) void k_fused_reduce_wave(FusedArgs A) {
  const int q = blockIdx.x * (kWG / 64) + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (q >= A.n_act) return;
  double sx = 0.0, sy = 0.0, sz = 0.0, sp = 0.0, qm = 0.0, sm = __builtin_inf();
  const int64_t stride = 6 * static_cast<int64_t>(A.n_act);
  for (int s = lane; s < A.plan.n_slices; s += 64) {
    const double *in = A.part + s * stride;
    sx += in[q];
    sy += in[A.n_act + q];
    sz += in[2 * A.n_act + q];
    sp += in[3 * A.n_act + q];
    qm = fmax(qm, in[4 * A.n_act + q]);
    sm = fmin(sm, in[5 * A.n_act + q]);
  }
  sx = wave_sum(sx);
  sy = wave_sum(sy);
  sz = wave_sum(sz);
  sp = wave_sum(sp);
  qm = wave_max(qm);
  sm = wave_min(sm);
  if (lane == 0) finish_all<V, NEWTON>(A, q, A.idx[q], sx, sy, sz, sp, qm, sm);
}

// Same, a workgroup per 64 consecutive targets whose kRowsWaves waves each combine a
// contiguous range of the slices in order, then the waves in order: the association of
// the force's k_force_reduce_rows, so the results stay those of the separate kernels.
template <class V, int NEWTON>
__global__ __launch_bounds__(64 * kRowsWaves) void k_fused_reduce_rows(FusedArgs A) {
  __shared__ double sums[kRowsWaves][6][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int q = blockIdx.x * 64 + lane;
  const int S = A.plan.n_slices;
  const int L = (S + kRowsWaves - 1) / kRowsWaves;
  const int s1 = min(S, (w + 1) * L);
  double t[6] = {0.0, 0.0, 0.0, 0.0, 0.0, __builtin_inf()};
  if (q < A.n_act) {
    const int64_t stride = 6 * static_cast<int64_t>(A.n_act);
#pragma unroll 4
    for (int s = w * L; s < s1; ++s) {
      const double *in = A.part + s * stride;
#pragma unroll
      for (int c = 0; c < 4; ++c) t[c] += in[c * A.n_act + q];
      t[4] = fmax(t[4], in[4 * A.n_act + q]);
      t[5] = fmin(t[5], in[5 * A.n_act + q]);
    }
  }
#pragma unroll
  for (int c = 0; c < 6; ++c) sums[w][c][lane] = t[c];
  __syncthreads();
  if (w == 0 && q < A.n_act) {
    double f[6] = {0.0, 0.0, 0.0, 0.0, 0.0, __builtin_inf()};
    for (int ww = 0; ww < kRowsWaves; ++ww) {
#pragma unroll
      for (int c = 0; c < 4; ++c) f[c] += sums[ww][c][lane];
      f[4] = fmax(f[4], sums[ww][4][lane]);
      f[5] = fmin(f[5], sums[ww][5][lane]);
    }
    finish_all<V, NEWTON>(A, q, A.idx[q], f[0], f[1], f[2], f[3], f[4], f[5]);
  }
}

template <class V, int NEWTON, int CH, int SH>
void launch_main(FusedArgs &A, hipStream_t st) {
  const dim3 grid(A.plan.nblk), block(kWG);
  if (A.pot)
    hipLaunchKernelGGL((k_fused<V, NEWTON, 1, CH, SH>), grid, block, 0, st, A);
  else
    hipLaunchKernelGGL((k_fused<V, NEWTON, 0, CH, SH>), grid, block, 0, st, A);
}

template <class V, int NEWTON>
hipError_t run(FusedArgs &A, int chunk, hipStream_t st) {
  if (A.share && chunk == kChunkTiny)
    launch_main<V, NEWTON, kChunkTiny, kShare>(A, st);
  else if (A.share && chunk == kChunkSmall)
    launch_main<V, NEWTON, kChunkSmall, kShare>(A, st);
  else if (A.share)
    launch_main<V, NEWTON, kTJ, kShare>(A, st);
  else if (chunk == kChunkSmall)
    launch_main<V, NEWTON, kChunkSmall, 1>(A, st);
  else
    launch_main<V, NEWTON, kTJ, 1>(A, st);
  // the force's choice for the same call
  if (force_rows_reduce(A.plan.n_slices, A.n_act, A.share != 0)) {
    const int nb = (A.n_act + 63) / 64;
    hipLaunchKernelGGL((k_fused_reduce_rows<V, NEWTON>), dim3(nb), dim3(64 * kRowsWaves), 0, st,
                       A);
  } else if (use_wave_reduce(A.plan.n_slices, A.n_act)) {
    const int nb = (A.n_act + kWG / 64 - 1) / (kWG / 64);
    hipLaunchKernelGGL((k_fused_reduce_wave<V, NEWTON>), dim3(nb), dim3(kWG), 0, st, A);
  } else {
    const int nb = (A.n_act + kWG - 1) / kWG;
    hipLaunchKernelGGL((k_fused_reduce<V, NEWTON>), dim3(nb), dim3(kWG), 0, st, A);
  }
  return hipGetLastError();
}

// The force's split of the same call.
SplitPlan fused_plan(const tsbts_ctx *c, int n_act, int *chunk, int *n_units, int *share) {
  const ShareShape sh = share_force(c, n_act);
  *share = sh.chunk != 0;
  *chunk = sh.chunk ? sh.chunk : scalar_chunk(c, n_act, 1);
  *n_units = sh.chunk ? sh.n_units : static_cast<int>(c->npad / *chunk);
  return sh.chunk ? sh.plan : plan_split(n_act, 1, *n_units, c->tune_blocks);
}

}  // namespace

// Small sets, whose lanes the fused pass would leave idle, and sets whose criterion over the
// spatial order saves more than the fused pass does.  Measured (us of device time, fused /
// apart): mixed N = 131072 k = 2500 282 / 302, 3000 321 / 323, 3500 364 / 342; 262144 2000 435 /
// 455, 2500 550 / 525; float64 32768 3500 159 / 163, 4095 178 / 170; 65536 2000 184 / 200, 2500
// 239 / 233; 131072 1500 288 / 305, 2000 351 / 320; 262144 1100 435 / 468, 1500 580 / 511.  In
// mixed precision few targets of very many particles also go apart: 64 of N = 131072 45.8 /
// 44.8, of 262144 76 / 68, 180 91 / 90.  Sets of 4096 targets or more stay in one pass.
bool criterion_apart(const tsbts_ctx *c, int n_act) {
  if (n_act <= kSmallAct) return true;
  if (!share_force(c, n_act).chunk) return false;
  const bool fp64 = c->precision == TSBTS_FP64;
  if (!fp64 && c->n >= 196608 && n_act <= 128) return true;
  return cells_criterion_applies(c, n_act) &&
         (fp64 ? c->n * (n_act - 900) >= 95000000 : c->n * (n_act - 1300) >= 260000000);
}

// Every small and shared set: the host applies the step rule and issues the next prediction
// while the force still runs, which is worth more than the separations evaluated twice.
// Native eras with the criterion first (ms, fused / apart): mixed N = 300 1.53 / 1.33, 1000
// 2.53 / 1.92, 4096 6.5 / 5.7, 16384 18.4 / 15.5; float64 4096 6.3 / 5.7, 16384 20.5 / 16.9; at N =
// 131072 the steps of 33 to 256 targets 75 / 52 of 460 ms, larger ones equal.
bool criterion_first(const tsbts_ctx *c, int n_act) {
  return n_act <= kSmallAct || share_force(c, n_act).chunk != 0;
}

int64_t fused_partials_needed(const tsbts_ctx *c, int n_act) {
  int chunk, n_units, share;
  return static_cast<int64_t>(fused_plan(c, n_act, &chunk, &n_units, &share).n_slices) * 6 *
         n_act;
}

hipError_t launch_fused(tsbts_ctx *c, const int32_t *idx, int n_act, double eta, double *acc,
                        double *pot, double *dtc, hipStream_t st, const CorrectArgs *corr) {
  FusedArgs A;
  A.n = c->n;
  A.npad = c->npad;
  A.p32 = c->p32;
  A.p64 = c->p64;
  A.v64 = c->v64;
  A.idx = idx;
  A.n_act = n_act;
  int chunk;
  A.plan = fused_plan(c, n_act, &chunk, &A.n_units, &A.share);
  A.eps2f = static_cast<float>(c->eps * c->eps);
  A.eps2 = c->eps * c->eps;
  A.eta = eta;
  A.part = c->part;
  A.acc = acc;
  A.pot = pot;
  A.dtc = dtc;
  A.correct = corr ? 1 : 0;
  if (corr) A.corr = *corr;
  if (c->precision == TSBTS_FP64) return run<Fp64, 0>(A, chunk, st);
  const bool sep64 = (c->flags & TSBTS_FLAG_HILO_SEPARATION) == 0;
  const bool newton = (c->flags & TSBTS_FLAG_NEWTON) != 0;
  if (sep64) return newton ? run<MixSep64, 1>(A, chunk, st) : run<MixSep64, 0>(A, chunk, st);
  return newton ? run<MixHiLo, 1>(A, chunk, st) : run<MixHiLo, 0>(A, chunk, st);
}

}  // namespace tsbts
