// Internal declarations of the TSBTS HIP library: the context, device helpers shared by
// the kernels, and the host-side launchers each kernel file provides.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/tsbts.h"

namespace tsbts {

constexpr int kWG = 256;    // threads per workgroup (4 wave64)
constexpr int kTJ = 256;    // j-particles per LDS tile
constexpr int kPad = 512;   // particle arrays are padded to a multiple of this
constexpr float kFarF = 1.0e18f;  // position of padding particles (zero mass)
constexpr double kFar = 1.0e18;

// Plane indices of the context's particle arrays.
//   p64: [5][npad] float64: x, y, z, m, w = m^(-2/3)
//   v64: [3][npad] float64: velocities at the predicted time
//   p32: [8][npad] float32: x_hi, y_hi, z_hi, m, x_lo, y_lo, z_lo, w = m^(-2/3)
enum { P64_X = 0, P64_M = 3, P64_W = 4, P64_PLANES = 5 };
enum { P32_XH = 0, P32_M = 3, P32_XL = 4, P32_W = 7, P32_VX = 8, P32_E = 11, P32_PLANES = 12 };
// History record state planes: r(3), v(3), a(3)
constexpr int kHistPlanes = 9;
constexpr int kDefaultBlocks = 8192;  // workgroups a split-j launch aims for

struct History {
  // records being appended during a pass
  int32_t *pid = nullptr, *rank = nullptr;
  double *t = nullptr, *s = nullptr;  // s: [9][cap]
  int64_t cap = 0, count = 0;
  bool recording = false;
  // finished pass, grouped by particle
  double *ht = nullptr, *hs = nullptr;  // hs: [9][hcap]
  int32_t *off = nullptr;               // [n + 1]
  int32_t *cur = nullptr;               // [n] interpolation cursor
  int64_t hcap = 0, hcount = 0;
  bool valid = false;
  int32_t *cnt = nullptr;               // [n] records per particle in the current pass
  int32_t *tsum = nullptr;              // per-tile sums of the offset scan
};

}  // namespace tsbts

struct tsbts_ctx {
  int64_t n = 0, npad = 0;
  double eps = 0.0;
  int precision = TSBTS_MIXED;
  int flags = 0;
  int device = 0;
  // bound caller state
  double *r = nullptr, *v = nullptr, *a = nullptr, *t_last = nullptr, *dt = nullptr;
  const double *m = nullptr;
  // predicted particle arrays
  double *p64 = nullptr, *v64 = nullptr;
  float *p32 = nullptr;
  double pred_t = 0.0;
  bool have_pred = false;
  // partial sums of split-j reductions
  double *part = nullptr;
  int64_t part_cap = 0;  // elements
  // adjoint seeds in particle order (all-active adjoint), [4][npad]
  double *gord = nullptr;
  // energy partials
  double *epart = nullptr;
  int64_t epart_cap = 0;
  tsbts::History h;
  // native host scheduler (tsbts_sched_*), owned
  void *sched = nullptr;
  // launch-shape tuning (tsbts_tune)
  int tune_blocks = tsbts::kDefaultBlocks;
  int tune_ipl = 0;
  int tune_chunk = 0;  // j-particles per split unit of the scalar-load kernels (0: automatic)
  int tune_sym = 2;    // symmetric all-targets kernels: 0 off, 1 on, 2 automatic
  int check_idx = 0;   // device range check of every active set (TSBTS_TUNE_CHECK_INDICES)
  int *idx_flag_h = nullptr, *idx_flag_d = nullptr;  // its results: [0] an index out of
                                                      // range, [1] a repeated index
                                                      // (mapped pinned memory)
  int32_t *idx_seen = nullptr;  // [n] occurrence counters of the check
  // finished-workgroup counts of the launches whose last workgroup reduces the partials
  // (last_workgroup_partials), zero between launches (force_done, step_done, share_done)
  uint32_t *done = nullptr;
  // symmetric all-targets kernels: work items (int4) and partials
  void *sym_items = nullptr;
  int sym_items_n = 0;
  int64_t sym_items_npad = 0;
  int sym_chunk = 0;
  void *sym_part = nullptr;
  int64_t sym_part_bytes = 0;
  // split calls of large partial active sets (split.hip): one allocation for the compact
  // copies of the targets and of the other particles (split_cap particles each), the
  // marks and scan of the other particles, the symmetric part's results and work items
  void *split_buf = nullptr;
  int64_t split_cap = 0;
  int tune_split = 2;  // 0 off, 1 from kSplitMinAct targets, 2 automatic
  // spatial order of the criterion of large active sets (timestep_cells.hip): one
  // allocation for npad particles, not tried again once it failed
  void *cell_buf = nullptr;
  bool cell_refused = false;
  char err[512] = {0};
};

namespace tsbts {

// ------------------------------------------------------------------ device helpers

// Workgroups are dispatched round-robin over the 8 XCDs (each with its own L2).  Renumber
// so that each XCD receives a contiguous range of logical block ids; nblk is a multiple
// of 8.
__device__ __forceinline__ int xcd_linear(int bid, int nblk) {
  return (bid & 7) * (nblk >> 3) + (bid >> 3);
}

// A wave-uniform value as a vector operand: a float32 instruction with a scalar register
// among its operands issues in 4.4 cycles, with vector registers only in 2.7 (measured at
// 8 waves per SIMD; float64 ones take 4.4 either way).
template <class T>
__device__ __forceinline__ T in_vector(T x) {
  asm("" : "+v"(x));
  return x;
}

__device__ __forceinline__ float rsq_f32(float x) { return __builtin_amdgcn_rsqf(x); }
__device__ __forceinline__ double rsq_f64_approx(double x) { return __builtin_amdgcn_rsq(x); }

// 1/sqrt(s) in float64 from the hardware estimate y and its residual e = 1 - s y^2 (at most
// 1.04e-7): y (1 + e/2 + 3 e^2/8), the next term below 1e-21.  Five operations where two
// Newton steps take seven, and nearer (1 - s y^2 at most 3.8e-16 against 5.3e-16, mean
// 7e-20 against 3e-17 over s = 2^-40 .. 2^40).  For s from 5.6e-309: below, y^2 overflows,
// where the Newton steps still gave the root (separations below 7.5e-155 without softening,
// whose accelerations overflow either way).
__device__ __forceinline__ double rsqrt_f64(double s) {
  const double y = rsq_f64_approx(s);
  const double e = fma(-s, y * y, 1.0);
  return fma(y * e, fma(0.375, e, 0.5), y);
}

// k s^(-3/2) likewise: k y^3 (1 + 3 e/2 + 15 e^2/8).  With POT also adds k s^(-1/2) to pot,
// in three operations, the last one the sum's (float64 with the potential, all of N = 32767:
// 738 -> 704 us, 16384 of 131072 1451 -> 1389; two Newton steps took 724 and 1426).
template <int POT>
__device__ __forceinline__ double scaled_inv_cube_f64(double s, double k, double &pot) {
  const double y = rsq_f64_approx(s);
  const double t = y * y;
  const double e = fma(-s, t, 1.0);
  const double ky = k * y;
  const double a = ky * t;
  if (POT) pot = fma(ky, fma(e, fma(0.375, e, 0.5), 1.0), pot);
  return fma(a * e, fma(1.875, e, 1.5), a);
}

// Split a float64 into a float32 pair whose sum carries ~48 significant bits.
__device__ __forceinline__ void split_hilo(double x, float &hi, float &lo) {
  hi = static_cast<float>(x);
  lo = static_cast<float>(x - static_cast<double>(hi));
}

// m^(-2/3): the per-source weight of the free-fall criterion term (infinite for m = 0).
__device__ __forceinline__ double ff_weight(double m) {
  return m > 0.0 ? 1.0 / cbrt(m * m) : __builtin_inf();
}

// Combination of lanes O apart (O = 32, 16, ..., 1) without LDS where the hardware has such
// a move: the halves and the odd and even rows of 16 lanes change places between two
// registers (v_permlane32_swap, v_permlane16_swap), lanes 8, 2 and 1 apart come as an
// operand (DPP row rotation and quad permutation); only 4 apart is an LDS swizzle.  A
// butterfly of ds_bpermute shuffles took 5 LDS round trips more.
// lane_fold: every lane with bit O clear gets op over both lanes' a, the others over b.
template <int O>
__device__ __forceinline__ int lane_move(int x) {
  if constexpr (O == 8) return __builtin_amdgcn_update_dpp(0, x, 0x128, 0xf, 0xf, true);
  else if constexpr (O == 4) return __builtin_amdgcn_ds_swizzle(x, 0x101f);
  else if constexpr (O == 2) return __builtin_amdgcn_update_dpp(0, x, 0x4e, 0xf, 0xf, true);
  else return __builtin_amdgcn_update_dpp(0, x, 0xb1, 0xf, 0xf, true);
}
template <int O>
__device__ __forceinline__ float lane_move(float x) {
  return __builtin_bit_cast(float, lane_move<O>(__builtin_bit_cast(int, x)));
}
template <int O>
__device__ __forceinline__ double lane_move(double x) {
  int2 v = __builtin_bit_cast(int2, x);
  v.x = lane_move<O>(v.x);
  v.y = lane_move<O>(v.y);
  return __builtin_bit_cast(double, v);
}
template <int O>
__device__ __forceinline__ void lane_swap(unsigned &a, unsigned &b) {
  static_assert(O == 32 || O == 16, "halves or rows");
  // two registers whatever the compiler knows of the values: the move writes both, and
  // equal operands were seen to be given one register
  asm("" : "+v"(b));
  if constexpr (O == 32) {
    const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
    a = r[0];
    b = r[1];
  } else {
    const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
    a = r[0];
    b = r[1];
  }
}
template <int O>
__device__ __forceinline__ void lane_swap(float &a, float &b) {
  unsigned u = __float_as_uint(a), v = __float_as_uint(b);
  lane_swap<O>(u, v);
  a = __uint_as_float(u);
  b = __uint_as_float(v);
}
template <int O>
__device__ __forceinline__ void lane_swap(double &a, double &b) {
  uint2 u = __builtin_bit_cast(uint2, a), v = __builtin_bit_cast(uint2, b);
  lane_swap<O>(u.x, v.x);
  lane_swap<O>(u.y, v.y);
  a = __builtin_bit_cast(double, u);
  b = __builtin_bit_cast(double, v);
}
template <int O, class T, class Op>
__device__ __forceinline__ T lane_fold(T a, T b, int lane, Op op) {
  if constexpr (O >= 16) {
    lane_swap<O>(a, b);
    return op(a, b);
  } else {
    // both read first: a select between array elements would become a select of
    // addresses, which keeps a float64 array out of registers
    const bool up = (lane & O) != 0;
    const T keep = up ? b : a;
    const T send = up ? a : b;
    return op(keep, lane_move<O>(send));
  }
}
// Every lane's x combined with that of the lane O apart.
template <int O, class T, class Op>
__device__ __forceinline__ T lane_pair(T x, Op op) {
  if constexpr (O >= 16) {
    T y = x;
    lane_swap<O>(x, y);
    return op(x, y);
  } else {
    return op(x, lane_move<O>(x));
  }
}

// Fixed-order butterfly reductions over one wave64 (every lane receives the result).
template <int O, class T, class Op>
__device__ __forceinline__ T wave_combine(T x, Op op) {
  x = lane_pair<O>(x, op);
  if constexpr (O > 1) x = wave_combine<O / 2>(x, op);
  return x;
}
__device__ __forceinline__ double wave_sum(double x) {
  return wave_combine<32>(x, [](double a, double b) { return a + b; });
}
__device__ __forceinline__ double wave_max(double x) {
  return wave_combine<32>(x, [](double a, double b) { return fmax(a, b); });
}
__device__ __forceinline__ double wave_min(double x) {
  return wave_combine<32>(x, [](double a, double b) { return fmin(a, b); });
}

// Reduction over one wave64 of NV values per lane (NV a power of two, at most 64) by
// recursive halving: at each of the log2(NV) stages a lane keeps half of its values and
// combines them with its partner's copies of the same values (63 moves for 64 values where
// separate butterflies take 384); the remaining stages combine the one value left across
// lanes.  Lane l returns value l >> (6 - log2 NV), combined over all 64 lanes (the same in
// every lane of its group); x is consumed.
template <int O, int NV, class T, class Op>
__device__ __forceinline__ void halve(T *x, int lane, Op op) {
  if constexpr (NV > 1) {
#pragma unroll
    for (int i = 0; i < NV / 2; ++i) x[i] = lane_fold<O>(x[i], x[NV / 2 + i], lane, op);
    if constexpr (O > 1) halve<O / 2, NV / 2>(x, lane, op);
  } else {
    x[0] = wave_combine<O>(x[0], op);
  }
}
template <int NV, class T, class Op>
__device__ __forceinline__ T wave_reduce_many(T (&x)[NV], int lane, Op op) {
  static_assert(NV >= 1 && NV <= 64 && (NV & (NV - 1)) == 0, "power of two up to 64");
  halve<32, NV>(x, lane, op);
  return x[0];
}

// Whether this workgroup is the last of `count` to get here, for a launch whose last
// workgroup finishes a reduction over the others' partials.  Everything it reads of theirs
// was written by store_partial and is read by load_partial: those pass the caches that the
// XCDs do not share (relaxed atomics of agent scope), so no cache is written back or
// emptied; every thread waits until its stores have arrived before one thread counts the
// workgroup in `done`.  The last one resets the count to zero for the next launch.  No
// workgroup waits for another.  Every thread of the workgroup must call it.  With the
// register moves above instead of LDS shuffles, small calls on N = 4096 took (us, force /
// criterion, before with agent-scope fences): 4 targets 7.0 / 8.0 -> 5.1 / 5.7, 16 targets
// 9.7 / 8.9 -> 7.3 / 6.9; one target, whose 64 mostly empty parts are no longer added,
// 8.7 / 10.3 -> 4.7 / 5.3.
__device__ __forceinline__ void store_partial(double *p, double x) {
  __hip_atomic_store(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ double load_partial(const double *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ bool last_workgroup_partials(uint32_t *done, uint32_t count) {
  __shared__ uint32_t last;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x == 0) {
    const uint32_t before = atomicAdd(done, 1u);
    last = before + 1 == count ? 1u : 0u;
    if (last) atomicExch(done, 0u);
  }
  __syncthreads();
  return last != 0;
}

// Split-j partials are combined by one thread per target when there are few slices and
// by one wave per target (lanes striding over the slices) when there are many.
constexpr int kWaveReduceSlices = 16;
// ... but only for few targets: with many targets one thread per target reads the
// partials coalesced, while one wave per target would touch a cache line per slice.
constexpr int64_t kWaveReduceMaxTargets = 4096;
__host__ __device__ inline bool use_wave_reduce(int n_slices, int64_t n_targets) {
  return n_slices >= kWaveReduceSlices && n_targets <= kWaveReduceMaxTargets;
}
// From kRowsReduceMinTargets targets on (force and criterion), many slices are combined
// by a workgroup per 64 consecutive targets instead, its kRowsWaves waves each adding a
// contiguous range of slices: rows of 64 consecutive partials are read coalesced (the
// wave-per-target form touches a cache line per 8-byte partial).  Below that there are
// too few such workgroups (at 256 targets 4, each wave walking 128 slices: 43 against
// 34 us per call at N = 131072).
// With at most kRowsFewSlices slices a wave walks few of them, and it pays from fewer
// targets on: always for the kernels whose waves share 64 targets, whose slices are that
// few; for the other forms from kRowsFewForce targets of the force (1500 of N = 16384, 64
// slices, 30.7 -> 27.8 us a call; 500 of N = 4096, 64 slices, 9.6 -> 10.4) and kRowsFewStep
// of the criterion (1500 28.4 -> 25.5, 500 12.5 -> 11.9), there from kRowsTinyStep where
// there are kRowsTinySlices at most (16 of N = 20011, 79 slices, 8.1 -> 7.9; of N = 32768,
// 128 slices, 8.1 -> 8.6)).  Few targets are one such workgroup, whose waves would walk all
// slices: one target's force at N = 60000, 235 slices, 5.1 us with a wave per target, 11.0
// with rows.
constexpr int64_t kRowsReduceMinTargets = 2048;
constexpr int kRowsWaves = 16;
constexpr int kRowsFewSlices = 256;
constexpr int kRowsFewForce = 1024, kRowsFewStep = 33;
constexpr int kRowsTinyStep = 4, kRowsTinySlices = 96;
__host__ __device__ inline bool use_rows_reduce(int n_slices, int64_t n_targets,
                                                int64_t few = kRowsReduceMinTargets) {
  return n_slices >= kWaveReduceSlices &&
         (n_targets >= kRowsReduceMinTargets ||
          (n_slices <= kRowsFewSlices && n_targets >= few));
}
__host__ __device__ inline bool force_rows_reduce(int n_slices, int64_t n_targets,
                                                  bool shared) {
  return use_rows_reduce(n_slices, n_targets, shared ? 1 : kRowsFewForce);
}
__host__ __device__ inline bool step_rows_reduce(int n_slices, int64_t n_targets,
                                                 bool shared) {
  return use_rows_reduce(n_slices, n_targets,
                         shared ? 1 : n_slices <= kRowsTinySlices ? kRowsTinyStep : kRowsFewStep);
}

// The small-set kernels' last workgroup reduces the partials (W values per slice) itself
// when the launch has at most kFuseSlices workgroups and each of its threads then reads
// at most kFuseLoads partials; otherwise a reduction kernel follows (512 workgroups, N =
// 131072, would leave the last one four times the loads in flight at a time).
constexpr int kFuseLoads = 32;
constexpr int kFuseSlices = 64;
__host__ __device__ inline bool fuse_small_reduce(int n_slices, int W) {
  const int parts = W <= kWG ? kWG / W : 1;
  return W <= kWG && n_slices <= kFuseSlices && (n_slices + parts - 1) / parts <= kFuseLoads;
}

// Tiles of kTJ that hold particles: the padding of the planes (to a multiple of kPad) can
// be a whole tile, which the kernels of few targets leave out.
inline int used_tiles(const tsbts_ctx *c) { return static_cast<int>((c->n + kTJ - 1) / kTJ); }

// Active sets up to this size use the j-parallel pair kernels (one source per lane).
constexpr int kSmallAct = 32;
// ... and for the float64 force kernel up to this size.
constexpr int kSmallActFp64 = 16;

__host__ __device__ constexpr int64_t round_up(int64_t x, int64_t q) {
  return (x + q - 1) / q * q;
}

// ------------------------------------------------------------------ launch plans

struct SplitPlan {
  int n_itiles;        // i-tiles of ipl*kWG targets
  int n_slices;        // j-slices
  int tiles_per_slice; // j-tiles of kTJ per slice
  int nblk;            // launched blocks (multiple of 8)
};

SplitPlan plan_split(int64_t n_targets, int ipl, int64_t n_jtiles, int target_blocks);

// Block -> (target tile, j-slice) of a split launch.  Each XCD takes a contiguous range of
// logical ids (xcd_linear).  When the slice count is a multiple of 8, each XCD's range is
// one group of n_slices/8 consecutive slices in which the slice varies fastest: the
// workgroups an XCD runs back to back share a target tile, whose gathered records then
// come from that XCD's L2, and sweep the group's slices, whose sources stay in the same
// L2.  Otherwise the target tile varies fastest over all slices.  Either way every
// (tile, slice) pair is computed by exactly one workgroup, as before the remapping.
__device__ __forceinline__ void split_tile(int bid, const SplitPlan &p, int &itile,
                                           int &slice) {
  const int L = xcd_linear(bid, p.nblk);
  const int g = (p.n_slices & 7) == 0 ? (p.n_slices >> 3) : 1;
  const int per = g * p.n_itiles;
  const int r = L % per;
  itile = r / g;
  slice = (L / per) * g + r % g;
}

// Targets per lane of the force and criterion kernels for an active set of n_act.
inline int targets_per_lane(const tsbts_ctx *c, int n_act) {
  if (c->tune_ipl) return c->tune_ipl;
  return n_act < 8192 ? 1 : 2;
}

// The force kernel reads its j-particles through wave-uniform (scalar) loads unless a
// targets-per-lane count was set, which selects the LDS-staged kernel.
inline bool force_scalar_j(const tsbts_ctx *c) { return c->tune_ipl == 0; }
// The automatic kernel form: a workgroup count, targets per lane or unit that was set keeps
// the forms it is defined for.
inline bool automatic_form(const tsbts_ctx *c) {
  return force_scalar_j(c) && c->tune_chunk == 0 && c->tune_blocks == kDefaultBlocks;
}
inline int force_targets_per_lane(const tsbts_ctx *c, int n_act) {
  return force_scalar_j(c) ? 1 : targets_per_lane(c, n_act);
}
// j-particles per split unit of the scalar-load kernels with a target per lane of the
// workgroup: whole tiles of kTJ, or quarter tiles when whole tiles would give too few
// workgroups to fill the chip, so that the j-range splits over 4x more workgroups.
constexpr int kChunkSmall = 64;
inline int scalar_chunk(const tsbts_ctx *c, int n_act, int ipl) {
  if (c->tune_chunk) return c->tune_chunk;
  const int64_t itiles = (n_act + ipl * kWG - 1) / (ipl * kWG);
  return itiles * (c->npad / kTJ) < 512 ? kChunkSmall : kTJ;
}
// Scalar-load kernels whose workgroup holds 64 targets, one per lane, and whose waves
// share the j-particles of a unit (kShare parts of `chunk`): for active sets below
// kShareMaxAct, where a target per lane of the workgroup leaves lanes without a target
// (33 targets in 256 lanes) and many slices for the reduction to read (472 of 64
// j-particles for 777 targets at N = 30011).  Measured (us, force / criterion, the other
// form first): mixed 64 targets N = 256 8.7 / 11.7 and 7.1 / 7.1, 1500 targets N = 4096
// 13.4 / 14.4 and 9.8 / 10.9, 777 targets N = 30011 36 / 33 and 21 / 24; float64 64
// targets N = 131072 39 / 45 and 23 / 24, 3000 targets N = 16384 45 / 54 and 41 / 46; from
// 4096 targets the other form is as fast or faster.  A tuned shape keeps the other form.
//   The j-particles per wave are the other form's chunk in the mixed force (its float32
// sums stay the same numbers; only float64 sums are regrouped), else 64, or 16 where
// units of 4 x 64 would be fewer than 512 workgroups.
constexpr int kShare = kWG / 64;
constexpr int kShareMaxAct = 4096;
constexpr int kShareTiles = kShareMaxAct / 64;
// With at most kShareFuse slices (few particles) the workgroup that finishes a tile of 64
// targets last reduces the tile's partials itself, in the order of the reduction kernels,
// instead of a second launch.  Block steps of 33 to 256 targets, in us (separate, fused):
// float64 N = 256 (4 slices) 26.8, 24.5, N = 500 (8) 29.3, 26.1; mixed N = 1000 (4, the
// criterion separate) 32.5, 32.1, with its 16 slices fused too 38.5; N = 4096 (16 and 64
// fused) 32.4, 40: more slices wait longer for the last one than a launch takes.  So few are
// N <= 512 in float64, N <= 2048 for the mixed force, and there N = 7681 to 8192 from 3841
// targets too, whose units are 256 j-particles per wave.
constexpr int kShareFuse = 8;
constexpr int kChunkTiny = 16;
struct ShareShape {
  int chunk;       // j-particles per wave and unit; 0: not this form
  int n_units;     // units of kShare * chunk (the last one may pass the padding)
  SplitPlan plan;  // n_itiles counts 64 targets
};
// Finished-workgroup counts: one for each launch that may overlap another on the context.
// The small-set force counts apart when its partials lie in another array than the
// context's (the fixed one), whose calls the caller need not order with the context's; the
// small-set criterion; then each tile of 64 targets of the force (which = 0) and the
// criterion (1).
constexpr int kDoneCounts = 3 + 2 * kShareTiles;
inline uint32_t *force_done(const tsbts_ctx *c, const double *part) {
  return c->done + (part == c->part ? 0 : 2);
}
inline uint32_t *step_done(const tsbts_ctx *c) { return c->done + 1; }
inline uint32_t *share_done(const tsbts_ctx *c, int which) {
  return c->done + 3 + which * kShareTiles;
}
// The split of n_cols j-particles for n_targets (chunk 0: 64, or 16 for few).
ShareShape share_split(int64_t n_targets, int64_t n_cols, int chunk);
int64_t share_partials_reserve(const tsbts_ctx *c);
// Parts of each of ntp tile pairs' sources in the energy, as a power of two (energy.hip).
int energy_part_bits(int64_t ntp);
int64_t gather_partials_reserve(const tsbts_ctx *c);
// Whether a call on this stream may allocate: not while the stream is captured, nor when
// that cannot be told (the legacy stream during another stream's capture).
bool may_allocate(hipStream_t st);
ShareShape share_force(const tsbts_ctx *c, int n_act);
ShareShape share_step(const tsbts_ctx *c, int n_act);
// The criterion kernel likewise for large active sets (from 8192 targets, two targets per
// lane, twice the workgroups).
inline bool criterion_scalar_j(const tsbts_ctx *c, int n_act) {
  return force_scalar_j(c) && (n_act >= 8192 || scalar_chunk(c, n_act, 1) == kChunkSmall);
}
inline int criterion_targets_per_lane(const tsbts_ctx *c, int n_act) {
  if (!criterion_scalar_j(c, n_act)) return targets_per_lane(c, n_act);
  return n_act >= 8192 ? 2 : 1;
}
inline int criterion_blocks(const tsbts_ctx *c, int n_act) {
  return criterion_scalar_j(c, n_act) && n_act >= 8192 ? 2 * c->tune_blocks : c->tune_blocks;
}

// ------------------------------------------------------------------ launchers
// Each returns a hipError_t from the launch (hipSuccess on success).

// New steps of the previous block step not yet stored (native scheduler; predict.hpp).
struct PendingSteps {
  const int64_t *tag;  // [n] (step << 32) | list position, written by the corrector
  const double *dt;    // [k] new steps, by position in that step's active list
  int64_t step;
  // the same steps as powers of two, dt[q] = 2^exp[q], when k <= kInlinePend (host
  // memory, copied into the launch arguments); null: the kernels read dt
  const int8_t *exp;
  int k;
};
struct InlineIdx;
hipError_t launch_predict(tsbts_ctx *c, double t_block, int use_history, hipStream_t st,
                          const PendingSteps *pend = nullptr, const InlineIdx *in = nullptr);
hipError_t launch_load_positions(tsbts_ctx *c, const double *r, const double *m,
                                 hipStream_t st);
hipError_t launch_snapshot(tsbts_ctx *c, double T, double *r_out, double *v_out,
                           hipStream_t st);

struct CorrectArgs;
// Force, potential and criterion (with the predicted velocities) in one pass; with corr,
// the corrector runs in its reduction.
int64_t fused_partials_needed(const tsbts_ctx *c, int n_act);
hipError_t launch_fused(tsbts_ctx *c, const int32_t *idx, int n_act, double eta, double *acc,
                        double *pot, double *dtc, hipStream_t st,
                        const CorrectArgs *corr = nullptr);
// Tags of the native scheduler's corrector: each target g gets tag[g] = (step << 32) | q.
struct StepTags {
  int64_t *tag;
  int64_t step;
};
int force_criterion_correct(tsbts_ctx *c, const int32_t *idx, int32_t n_act, double t_block,
                            double eta, double *acc, double *dtc, hipStream_t stream,
                            const StepTags *tags = nullptr);
// Force on the active set and its corrector in the same launches (checked like the two
// entry points; returns a status code).  With `in`, the active list arrives by value
// and the first kernel writes it to idx (which must then not be checked beforehand).
// With dtc, also the criterion (eta) of the corrected targets when small_criterion_fused
// holds; *crit_done tells whether it did (else the caller runs tsbts_timestep).
int force_correct_predicted(tsbts_ctx *c, const int32_t *idx, int32_t n_act, double t_block,
                            int use_history, double *acc, hipStream_t stream,
                            const StepTags *tags = nullptr,
                            const PendingSteps *pend = nullptr,
                            const InlineIdx *in = nullptr, double eta = 0.0,
                            double *dtc = nullptr, int *crit_done = nullptr);
int force_correct(tsbts_ctx *c, const int32_t *idx, int32_t n_act, double t_block,
                  double *acc, hipStream_t stream, const StepTags *tags = nullptr);
// tsbts_predict with pending new steps and an inline active list (either may be null).
int predict_pending(tsbts_ctx *c, double t_block, int use_history, const PendingSteps *pend,
                    const InlineIdx *in, hipStream_t stream);
// With corr, every target's corrector (correct_one) runs where its force is final.
hipError_t launch_force(tsbts_ctx *c, const int32_t *idx, int n_act, double *acc,
                        double *pot, hipStream_t st, const CorrectArgs *corr = nullptr);
// Sources of a gather launch other than the context's predicted arrays (the second part
// of a split call): n particles that exclude every target (no self pair), padded to npad,
// planes laid out as the predicted arrays with stride npad; and the first part's results
// for each target, combined with the gather's where the target is finished: for the force
// [4][n_act] acceleration (x, y, z) and potential to add, for the criterion [2][n_act] the
// maximum of q and the minimum of s*w.
struct GatherSrc {
  const float *p32;   // [12][npad] or null (float64 mode)
  const double *p64;  // [5][npad]
  const double *v64;  // [3][npad]
  int64_t n, npad;
  const double *add;
};
// The gather force kernels (never the symmetric ones) with split-j partials in `part`
// and a split aiming for `blocks` workgroups; with `src`, its sources (always the
// scalar-load kernel).
hipError_t launch_force_gather(tsbts_ctx *c, const int32_t *idx, int n_act, double *acc,
                               double *pot, double *part, int blocks, hipStream_t st,
                               const CorrectArgs *corr = nullptr,
                               const GatherSrc *src = nullptr);
// float64 partials of that launch (0 when the j-range is not split).
int64_t force_partial_elems(const tsbts_ctx *c, int n_act, int blocks);
// Fixed partial-sum array of tsbts_force_noalloc: find its address on `device` (once per
// device); returns the HIP status of the lookup.
hipError_t noalloc_setup(int device);
// Its looked-up address on `device` (NULL before noalloc_setup succeeded there).
double *noalloc_partials(int device);
hipError_t launch_timestep(tsbts_ctx *c, const int32_t *idx, int n_act, double eta,
                           double *dtc, hipStream_t st);
// The gather criterion kernels with the sources `src` (the scalar-load kernel).
hipError_t launch_timestep_gather(tsbts_ctx *c, const int32_t *idx, int n_act, double eta,
                                  double *dtc, hipStream_t st, const GatherSrc *src);
// Split calls (split.hip): a large partial active set whose pairs among the targets are
// evaluated once for both (symmetric kernels on a compact copy of the targets) and whose
// pairs with the other particles by the gather kernels (a compact copy of those as
// sources).  split_applies: whether it serves a call of n_act targets; split_prepare
// allocates its buffers (host set-up; returns a status); the launches return
// hipErrorNotReady, with nothing launched, when the buffers are not there.
bool split_applies(const tsbts_ctx *c, int64_t n_act);
int split_prepare(tsbts_ctx *c, int64_t n_act);
hipError_t launch_force_split(tsbts_ctx *c, const int32_t *idx, int n_act, double *acc,
                              double *pot, hipStream_t st, const CorrectArgs *corr);
hipError_t launch_timestep_split(tsbts_ctx *c, const int32_t *idx, int n_act, double eta,
                                 double *dtc, hipStream_t st);
// Exclusive scan of cnt[0 .. n) into off[0 .. n] (off[n]: the total) with tile sums in
// tsum (one per 8192 counts); cur receives a copy of off[0 .. n) (may equal off).
hipError_t launch_exclusive_scan(const int32_t *cnt, int64_t n, int32_t *tsum, int32_t *off,
                                 int32_t *cur, hipStream_t st);
constexpr int64_t kScanCounts = 8192;  // counts per tile sum of launch_exclusive_scan
hipError_t launch_backward(tsbts_ctx *c, const int32_t *idx, int n_act, const double *ga,
                           const double *gp, double *gr, double *gm, hipStream_t st);
hipError_t launch_energy(tsbts_ctx *c, const double *r, const double *v, const double *m,
                         double *out, hipStream_t st);

hipError_t launch_correct(tsbts_ctx *c, const int32_t *idx, int n_act, double t_block,
                          const double *acc_new, hipStream_t st);
hipError_t launch_set_dt(tsbts_ctx *c, const int32_t *idx, int n_act, const double *dt_new,
                         hipStream_t st);
hipError_t launch_history_begin(tsbts_ctx *c, hipStream_t st);
hipError_t launch_history_end(tsbts_ctx *c, hipStream_t st);
hipError_t launch_leapfrog_adjoint(tsbts_ctx *c, int phase, double h, const double *rbar,
                                   double *vbar, double *abar, double *g_out,
                                   hipStream_t st);
// x[0 .. len) = v with a fill kernel (no memset node if a caller captures the stream).
hipError_t launch_fill(double *x, int64_t len, double v, hipStream_t st);
hipError_t launch_block_adjoint(tsbts_ctx *c, int phase, const int32_t *idx, int n_act,
                                double t_block, double *rbar, double *vbar, double *abar,
                                double *pbar, double *seeds, hipStream_t st);
// Largest active set of the j-parallel small-set kernels.
int small_act_limit(const tsbts_ctx *c);
// Predictor and force (with the corrector, if corr) in the small-set kernels, the sources
// predicted as they are loaded (n_act <= small_act_limit).
// With dtc (and corr), when small_criterion_fused holds, the launch's last workgroup also
// takes the criterion of the corrected targets into dtc (as launch_timestep would).
hipError_t launch_force_predicted(tsbts_ctx *c, const int32_t *idx, int n_act, double t_block,
                                  int use_history, double *acc, double *pot, hipStream_t st,
                                  const CorrectArgs *corr, const PendingSteps *pend = nullptr,
                                  const InlineIdx *in = nullptr, double eta = 0.0,
                                  double *dtc = nullptr);
// Whether launch_force_predicted takes the criterion of n_act targets itself: launches of
// one workgroup.
bool small_criterion_fused(const tsbts_ctx *c, int n_act);
// Whether a combined force + criterion call runs the criterion's and the force's own kernels
// instead of the fused pass (fused.hip).
bool criterion_apart(const tsbts_ctx *c, int n_act);
// The same for the native scheduler's step, whose host waits for the criterion alone.
bool criterion_first(const tsbts_ctx *c, int n_act);
// Symmetric all-targets criterion (timestep_sym.hip); plan from sym_plan.  With `set`, the
// kernels run on that particle set instead of the context's predicted arrays; with `raw`,
// each target's maximum and minimum go there unfinished ([2][n_act]) instead of to dtc.
struct SymPlan;
struct SymSet;
hipError_t launch_timestep_sym(tsbts_ctx *c, const SymPlan &plan, const int32_t *idx,
                               int n_act, double eta, double *dtc, hipStream_t st,
                               const SymSet *set = nullptr, double *raw = nullptr);
// Symmetric all-targets force (force_sym.hip): whether it serves the call, and its launch
// (on `set` instead of the context's predicted arrays when given).
bool force_sym_applies(const tsbts_ctx *c, int64_t n_act);
hipError_t launch_force_sym(tsbts_ctx *c, const SymPlan &plan, const int32_t *idx, int n_act,
                            double *acc, double *pot, hipStream_t st,
                            const CorrectArgs *corr, const SymSet *set = nullptr);
// Symmetric all-targets force adjoint (backward_sym.hip), after the seeds are ordered (gp:
// whether the potential has any).
bool bwd_sym_applies(const tsbts_ctx *c, int64_t n_act);
hipError_t launch_bwd_sym(tsbts_ctx *c, const SymPlan &plan, bool gp, double *gr, double *gm,
                          hipStream_t st);
// Adjoints of the passes of an era (hist_adjoint.hip).
hipError_t launch_interp_adjoint(tsbts_ctx *c, double t_block, double *pbar, double *hbar,
                                 hipStream_t st);
hipError_t launch_record_adjoint(tsbts_ctx *c, const int32_t *idx, int n_act, double t_block,
                                 const int32_t *off, const double *ht, int64_t n_records,
                                 const double *hbar, double *rbar, double *vbar,
                                 hipStream_t st);
hipError_t launch_accumulate3(int64_t len, const double *x0, const double *x1,
                              const double *x2, double *y0, double *y1, double *y2,
                              hipStream_t st);

// Free the native scheduler attached to a context (if any).
void destroy_scheduler(tsbts_ctx *c);

// Scratch needed by the split-j kernels for a given active-set size (float64 elements).
int64_t partial_elems_needed(const tsbts_ctx *c, int n_act);
int64_t energy_partials_needed(const tsbts_ctx *c);

}  // namespace tsbts
