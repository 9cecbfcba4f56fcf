// Time-step criterion (Eq. nbdt of Section 2) of a large active set over the spatial order
// of cells.hpp.  Per target the criterion keeps max |v_ij|^2 / |r_ij|^2 and
// min s m_j^(-2/3); both are decided by near particles, and a tile of 64 particles whose
// bounding box is far enough away cannot change either.  With D the distance between a
// target and a tile's box, every particle of the tile has
//   |v_ij|^2 / |r_ij|^2 <= (|v_i| + V)^2 / D^2   and   s m_j^(-2/3) >= (D^2 + eps^2) W
// (V the largest speed, W the smallest weight in the tile), so the tile is left out when
// the target's maximum and minimum so far are at least as good as both.  The pairs that
// are evaluated are the gather kernels' (pair_step); maxima and minima are exact, so the
// results equal theirs bit for bit, whatever the order.
//
// What bounds it: latency.  In a Plummer sphere a target needs about ten tiles (640 of
// 131072 particles), found through one test of a tile per lane against the box of
// kGroup = 16 consecutive targets of the order and one of each target against the tiles
// left; so few pairs remain that the loads between the tests, and the six launches of the
// sort, take most of the time.  A workgroup serves the group, its waves sharing the tiles
// and the bounds found (one wave per group: 545 us for all of 131072 targets, 154 of them
// in the slowest group).  In the pairs a tile's particle is on a lane and a target is
// wave-uniform (scalar loads, one target ahead); only targets whose own bounds the tile
// may change take part (a third of those of the visited tiles).
// Measured, all targets at N = 131072: 372 us mixed, 453 us float64, where the symmetric
// all-targets kernel takes 4335 and 8794; 40000 targets 205 us (1900 before).  With every
// particle in one point or line 740 and 1060 us.
#include "cells.hpp"
#include "criterion.hpp"

namespace tsbts {
namespace {

constexpr int kGroup = 16;     // targets of a workgroup
// Computed squares and bounds are off by a few float32 roundings: the distance is taken
// smaller and the speed larger by far more than those.
constexpr float kNear = 0.9999f, kFast = 1.0001f;
// Coordinates about the origin of the order rounded to float32 move by less than kUlps of
// their size; a float32 hi/lo pair is off by less than kPair of the coordinate itself.
constexpr float kUlps = 1.2e-7f, kPair = 1.5e-14f;

// A target: its side of the pairs, place among the particles, and place in the list.
template <class V>
struct __align__(64) Target {
  typename StepRec<V>::I i;
  int32_t place, q;
};

// A tile's box, largest speed and smallest weight.
template <class F>
struct __align__(sizeof(F) * 4) TileBox {
  F lo[3], hi[3], vmax, wmin;
};

// The sorted particles, read by load_jv.
struct CellArgs {
  const float *p32;
  const double *p64;
  const double *v64;
  int64_t npad;  // plane stride of the sorted copy
  int64_t n;
  int n_tiles;
  const double *origin;  // of positions and velocities in the tests
  const void *targets, *boxes;
  int n_act;
  double eps2, eta;
  double *dtc;
};

template <class F>
__device__ __forceinline__ F big() {
  if constexpr (sizeof(F) == 4) return __builtin_inff();
  else return __builtin_inf();
}

struct ScatterArgs {
  CellSort s;
  const double *p64, *v64;  // the predicted arrays
  const float *p32;
  int64_t npad, n;
  const int32_t *idx;
  int n_act;
  double *q64, *w64;  // the sorted copy (plane stride cap)
  float *q32;
  int64_t cap;
  void *targets;
};

// Thread t: particle t to its place in the sorted copy (the planes the policy reads), and
// target t to its place in the sorted targets.
template <class V>
__global__ __launch_bounds__(kWG) void k_cell_scatter(ScatterArgs a) {
  const int64_t t = static_cast<int64_t>(blockIdx.x) * kWG + threadIdx.x;
  if (t < a.n) {
    const int64_t d = cell_place(a.s, t), P = a.npad, Q = a.cap;
#pragma unroll
    for (int c = 0; c < 3; ++c) a.q64[c * Q + d] = a.p64[c * P + t];
    if constexpr (sizeof(typename V::F) == 4) {
      constexpr bool hilo = sizeof(typename V::I) == 6 * sizeof(float);
#pragma unroll
      for (int c = 0; c < P32_PLANES; ++c) {
        const bool used = c >= P32_W || (hilo && c != P32_M);
        if (used) a.q32[c * Q + d] = a.p32[c * P + t];
      }
    } else {
      a.q64[P64_W * Q + d] = a.p64[P64_W * P + t];
#pragma unroll
      for (int c = 0; c < 3; ++c) a.w64[c * Q + d] = a.v64[c * P + t];
    }
  }
  if (t < a.n_act) {
    const int64_t g = a.idx[t];
    struct { const float *p32; const double *p64, *v64; int64_t npad; } src{a.p32, a.p64, a.v64,
                                                                            a.npad};
    Target<V> r;
    r.i = load_iv<V>(src, g);
    r.place = cell_place(a.s, g);
    r.q = static_cast<int32_t>(t);
    const int d = cell_target_place(a.s, static_cast<int>(t), g);
    Target<V> *to = static_cast<Target<V> *>(a.targets);
    to[d] = r;
    if (d == a.n_act - 1)  // copies of the last target up to a whole group
      for (int e = a.n_act; e % kGroup != 0; ++e) to[e] = r;
  }
}

// Coordinate c of a target.
__device__ __forceinline__ double coord(const MixHiLo::I &i, int c) {
  return c == 0 ? static_cast<double>(i.xh) + i.xl
                : c == 1 ? static_cast<double>(i.yh) + i.yl : static_cast<double>(i.zh) + i.zl;
}
template <class I>
__device__ __forceinline__ double coord(const I &i, int c) {
  return c == 0 ? i.x : c == 1 ? i.y : i.z;
}

// Bounds of a coordinate about the origin o.
template <class F>
__device__ __forceinline__ void coord_bounds(double x, double o, F &lo, F &hi) {
  const F p = static_cast<F>(x - o);
  const F e = fma(fabs(p), F(kUlps), static_cast<F>(fabs(x)) * F(kPair));
  lo = p - e;
  hi = p + e;
}

// Speed about the reference velocity of a particle whose velocity the pairs see as v.
template <class F>
__device__ __forceinline__ F speed(const double *o, F vx, F vy, F vz) {
  const F x = static_cast<F>(static_cast<double>(vx) - o[3]);
  const F y = static_cast<F>(static_cast<double>(vy) - o[4]);
  const F z = static_cast<F>(static_cast<double>(vz) - o[5]);
  return sqrt(fma(x, x, fma(y, y, z * z)));
}

// A wave per tile: its box (rounded outwards), largest speed, smallest weight.
template <class V>
__global__ __launch_bounds__(kWG) void k_cell_boxes(CellArgs A) {
  using F = typename V::F;
  const int tile = blockIdx.x * (kWG / 64) + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (tile >= A.n_tiles) return;
  const int64_t j = static_cast<int64_t>(tile) * kCellTile + lane;
  F x[8];  // maxima: -lo, hi, speed, -weight
#pragma unroll
  for (int c = 0; c < 8; ++c) x[c] = -big<F>();
  if (j < A.n) {
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      coord_bounds<F>(A.p64[c * A.npad + j], A.origin[c], x[c], x[3 + c]);
      x[c] = -x[c];
    }
    const int64_t P = A.npad;
    if constexpr (sizeof(F) == 4) {
      const float *v = A.p32 + P32_VX * P + j;
      x[6] = speed<F>(A.origin, v[0], v[P], v[2 * P]);
      x[7] = -A.p32[P32_W * P + j];
    } else {
      const double *v = A.v64 + j;
      x[6] = speed<F>(A.origin, v[0], v[P], v[2 * P]);
      x[7] = -A.p64[P64_W * P + j];
    }
  }
  const F r = wave_reduce_many<8>(x, lane, [](F a, F b) { return fmax(a, b); });
  // lane l holds value l >> 3
  const int v = lane >> 3;
  if ((lane & 7) == 0)
    static_cast<F *>(const_cast<void *>(A.boxes))[tile * 8 + v] = v < 3 || v == 7 ? -r : r;
}

// Whether a tile may still change the maximum q or the minimum s of a target (or of any
// in a box [lo, hi] with speeds up to vel).  Written so that anything that is not a number
// keeps the tile; an overflowing distance means an overflowing |r_ij|^2.
template <class F>
__device__ __forceinline__ bool may_change(const TileBox<F> &b, const F (&lo)[3],
                                           const F (&hi)[3], F vel, F eps2, F q, F s) {
  F d2 = F(0);
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const F d = fmax(fmax(b.lo[c] - hi[c], lo[c] - b.hi[c]), F(0));
    d2 = fma(d, d, d2);
  }
  d2 *= F(kNear);
  const F u = (vel + b.vmax) * F(kFast);
  return !(u * u <= q * d2 && (d2 + eps2) * b.wmin * F(kNear) >= s);
}

// A target's record as the 16 registers of one wave-uniform (scalar) load.
typedef int TargetWords __attribute__((ext_vector_type(16)));
template <class V>
__device__ __forceinline__ TargetWords load_words(const Target<V> *t) {
  static_assert(sizeof(Target<V>) == sizeof(TargetWords), "one load");
  return *reinterpret_cast<const TargetWords *>(t);
}

// Maximum over the wave (DPP: lane shifts within rows of 16, then the rows' last lanes
// passed on; 6 short steps where a butterfly through LDS takes 6 round trips).
template <int CTRL, int ROWS, class F>
__device__ __forceinline__ F dpp_max(F x) {
  F y;
  if constexpr (sizeof(F) == 4) {
    const int v = __builtin_bit_cast(int, x);
    y = __builtin_bit_cast(F, __builtin_amdgcn_update_dpp(v, v, CTRL, ROWS, 0xf, false));
  } else {
    const int2 v = __builtin_bit_cast(int2, x);
    int2 w;
    w.x = __builtin_amdgcn_update_dpp(v.x, v.x, CTRL, ROWS, 0xf, false);
    w.y = __builtin_amdgcn_update_dpp(v.y, v.y, CTRL, ROWS, 0xf, false);
    y = __builtin_bit_cast(F, w);
  }
  return fmax(x, y);
}
__device__ __forceinline__ float lane_value(float x, int lane) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), lane));
}
__device__ __forceinline__ double lane_value(double x, int lane) {
  int2 v = __builtin_bit_cast(int2, x);
  v.x = __builtin_amdgcn_readlane(v.x, lane);
  v.y = __builtin_amdgcn_readlane(v.y, lane);
  return __builtin_bit_cast(double, v);
}
template <class F>
__device__ __forceinline__ F wave_max_dpp(F x) {
  x = dpp_max<0x111, 0xf>(x);  // row_shr:1, 2, 4, 8: lane 15 of each row has its row's
  x = dpp_max<0x112, 0xf>(x);
  x = dpp_max<0x114, 0xf>(x);
  x = dpp_max<0x118, 0xf>(x);
  x = dpp_max<0x142, 0xa>(x);  // row_bcast:15 into rows 1 and 3, row_bcast:31 into 2 and 3
  x = dpp_max<0x143, 0xc>(x);
  return lane_value(x, 63);
}

// Non-negative values as the unsigned integers that order like them.
__device__ __forceinline__ uint32_t bits(float x) { return __float_as_uint(x); }
__device__ __forceinline__ unsigned long long bits(double x) {
  return static_cast<unsigned long long>(__double_as_longlong(x));
}
__device__ __forceinline__ float value(uint32_t x) { return __uint_as_float(x); }
__device__ __forceinline__ double value(unsigned long long x) {
  return __longlong_as_double(static_cast<long long>(x));
}

// The tile's 64 particles against the targets of the group in `live` (a bit each).  Few
// tiles improve a bound, so the pairs' values are only compared with the target's; when
// some lane's are better, they are combined over the wave and kept in the lanes of the
// target and for the other waves.
template <class V, int MASK, class U>
__device__ __forceinline__ void tile_pairs(const CellArgs &A, const Target<V> *tg, int tile,
                                           uint32_t live, int lane, typename V::F eps2,
                                           U (*best)[kGroup], typename V::F &Q,
                                           typename V::F &S) {
  using F = typename V::F;
  const int j = tile * kCellTile + lane;
  const int n = static_cast<int>(A.n);
  const typename StepRec<V>::J J = load_jv<V>(A, MASK ? min(j, n - 1) : j);
  int t = __builtin_ctz(live);
  TargetWords words = load_words<V>(tg + t);
  while (live) {
    live &= live - 1;
    const int next = live ? __builtin_ctz(live) : t;
    const Target<V> T = __builtin_bit_cast(Target<V>, words);
    words = load_words<V>(tg + next);  // one target ahead of the pairs
    F q = F(0), s = big<F>();
    pair_step(T.i, J, eps2, MASK && (j >= n || j == T.place), q, s);
    if (__ballot(int(q > lane_value(Q, t)) | int(s < lane_value(S, t)))) {
      const F m = wave_max_dpp(q), l = -wave_max_dpp(-s);
      if ((lane & (kGroup - 1)) == t) {
        Q = fmax(Q, m);
        S = fmin(S, l);
      }
      // (a target's values are not negative: squares and weights are not)
      if (lane == 0) {
        atomicMax(&best[0][t], bits(m));
        atomicMin(&best[1][t], bits(l));
      }
    }
    t = next;
  }
}

// A workgroup per group of kGroup targets; its waves share the tiles (tile i to wave
// i % kWaves) and, through LDS, the targets' maxima and minima.  Lane l stands for target
// l % kGroup where bounds are kept and tested; in the pairs every target is uniform and
// lane l is particle l of the tile.
constexpr int kWaves = kWG / 64;

template <class V>
__global__ __launch_bounds__(kWG) void k_timestep_cells(
    CellArgs A0, const float *__restrict__ p32, const double *__restrict__ p64,
    const double *__restrict__ v64, const Target<V> *__restrict__ targets,
    const TileBox<typename V::F> *__restrict__ boxes, double *__restrict__ dtc) {
  using F = typename V::F;
  using U = decltype(bits(F(0)));
  __shared__ U best[2][kGroup];  // the targets' maxima and minima so far, as bits
  CellArgs A = A0;
  A.p32 = p32;
  A.p64 = p64;
  A.v64 = v64;
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int first = blockIdx.x * kGroup;
  const Target<V> *tg = targets + first;
  const F eps2 = static_cast<F>(A.eps2);
  const F inf = big<F>();
  if (threadIdx.x < kGroup) {
    best[0][threadIdx.x] = bits(F(0));
    best[1][threadIdx.x] = bits(inf);
  }
  __syncthreads();
  // the lane's target and its box, the group's box
  F lo[3], hi[3], glo[3], ghi[3], vel, gvel;
  int place;
  {
    const Target<V> mine = tg[lane & (kGroup - 1)];
    place = mine.place;
    vel = speed<F>(A.origin, mine.i.vx, mine.i.vy, mine.i.vz);
    F x[8];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      coord_bounds<F>(coord(mine.i.p, c), A.origin[c], lo[c], hi[c]);
      x[c] = -lo[c];
      x[3 + c] = hi[c];
    }
    x[6] = vel;
    x[7] = F(0);
    const F r = wave_reduce_many<8>(x, lane, [](F a, F b) { return fmax(a, b); });
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      glo[c] = -__shfl(r, 8 * c, 64);
      ghi[c] = __shfl(r, 8 * (3 + c), 64);
    }
    gvel = __shfl(r, 48, 64);
  }
  // The tiles that hold the group's particles come first, for good bounds: with their
  // neighbours when the group is compact, else those among the first 64 from the lowest.
  int pl = place, ph = place;
#pragma unroll
  for (int o = kGroup / 2; o >= 1; o >>= 1) {
    pl = min(pl, __shfl_xor(pl, o, 64));
    ph = max(ph, __shfl_xor(ph, o, 64));
  }
  pl = __builtin_amdgcn_readfirstlane(pl) / kCellTile;
  ph = __builtin_amdgcn_readfirstlane(ph) / kCellTile;
  int base = pl;      // tile of bit 0 of the mask below
  uint64_t own = 0;   // the tiles evaluated first
  if (ph - pl < 6) {
    base = max(pl - 1, 0);
    own = (uint64_t(1) << (min(ph + 1, A.n_tiles - 1) - base + 1)) - 1;
  } else {
#pragma unroll 1
    for (int t = 0; t < kGroup; ++t) {
      const int b = __builtin_amdgcn_readlane(place, t) / kCellTile - base;
      if (b < 64) own |= uint64_t(1) << b;
    }
  }
  // bounds of the lane's target and of the group
  F Q = F(0), S = inf, gq = F(0), gs = inf;
  // Pass -1: the wave's share of the group's own tiles.  Then chunks of 64 of the wave's
  // tiles, from the group's own outwards: a tile per lane against the group's box, and of
  // those left four at a time against each target.
  const int n_chunks = (A.n_tiles + 64 * kWaves - 1) / (64 * kWaves);
  const int c0 = ((pl + ph) / 2) / (64 * kWaves);
  const uint64_t stride4 = 0x1111111111111111ull;  // every kWaves-th bit
  static_assert(kWaves == 4, "stride4");
#pragma unroll 1
  for (int i = -1; i < n_chunks; ++i) {
    int from = base, step = 1;
    uint64_t todo = own & (stride4 << ((wv - base) & (kWaves - 1)));
    if (i >= 0) {
      int ch = c0 + ((i & 1) ? (i + 1) / 2 : -(i / 2));
      if (ch < 0) ch += n_chunks;
      if (ch >= n_chunks) ch -= n_chunks;
      from = ch * 64 * kWaves + wv;
      step = kWaves;
      const int tl = from + lane * kWaves;
      const int b = tl - base;
      bool live = tl < A.n_tiles && !(b >= 0 && b < 64 && ((own >> b) & 1));
      if (live) live = may_change(boxes[tl], glo, ghi, gvel, eps2, gq, gs);
      todo = __ballot(live);
    }
#pragma unroll 1
    while (todo) {
      int tile[4], cnt = 0;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        // (past the last one: the wave's first tile, which exists when todo had a bit)
        tile[u] = todo ? from + __builtin_ctzll(todo) * step : tile[0];
        cnt += todo ? 1 : 0;
        todo &= todo - 1;
      }
      uint64_t hit = ~uint64_t(0);
      if (i >= 0) {  // lanes of quarter u test tile u
        const int u = lane / kGroup;
        const int tu = u == 0 ? tile[0] : u == 1 ? tile[1] : u == 2 ? tile[2] : tile[3];
        hit = __ballot(may_change(boxes[tu], lo, hi, vel, eps2, Q, S));
      }
#pragma unroll 1
      for (int w = 0; w < cnt; ++w) {
        uint32_t live = static_cast<uint32_t>(hit) & ((1u << kGroup) - 1);
        hit >>= kGroup;
        const int tw = tile[0];
        tile[0] = tile[1];
        tile[1] = tile[2];
        tile[2] = tile[3];
        if (!live) continue;
        if ((tw >= pl && tw <= ph) || tw + 1 == A.n_tiles)
          tile_pairs<V, 1>(A, tg, tw, live, lane, eps2, best, Q, S);
        else
          tile_pairs<V, 0>(A, tg, tw, live, lane, eps2, best, Q, S);
      }
    }
    if (i < 0) __syncthreads();
    // whatever the other waves have found by now serves as well
    const int t = lane & (kGroup - 1);
    Q = value(*static_cast<volatile U *>(&best[0][t]));
    S = value(*static_cast<volatile U *>(&best[1][t]));
    gq = Q;
    gs = S;
#pragma unroll
    for (int o = kGroup / 2; o >= 1; o >>= 1) {
      gq = fmin(gq, __shfl_xor(gq, o, 64));
      gs = fmax(gs, __shfl_xor(gs, o, 64));
    }
  }
  __syncthreads();
  if (threadIdx.x < kGroup && first + lane < A.n_act)
    dtc[tg[lane].q] = finish_dt(A.eta, value(best[0][lane]), value(best[1][lane]));
}

// The device arrays of one call, carved from the context's buffer (base = null: its size).
struct CellBufs {
  CellSort sort;
  double *q64, *w64;
  float *q32;
  void *targets, *boxes;
};

int64_t cell_layout(const tsbts_ctx *c, char *base, CellBufs *b) {
  const int64_t cap = c->npad;
  int64_t o = 0;
  auto take = [&](int64_t bytes) {
    char *p = base ? base + o : nullptr;
    o += round_up(bytes, 256);
    return p;
  };
  const bool mixed = c->precision == TSBTS_MIXED;
  b->sort.origin = reinterpret_cast<double *>(take(6 * sizeof(double)));
  b->sort.planes = reinterpret_cast<float *>(take(3 * kCellSide * sizeof(float)));
  b->sort.count = reinterpret_cast<int32_t *>(take(2 * kCells * sizeof(int32_t)));
  b->sort.key = reinterpret_cast<int32_t *>(take(cap * sizeof(int32_t)));
  b->sort.rank = reinterpret_cast<int32_t *>(take(cap * sizeof(int32_t)));
  b->sort.trank = reinterpret_cast<int32_t *>(take(cap * sizeof(int32_t)));
  b->q64 = reinterpret_cast<double *>(take(P64_PLANES * cap * sizeof(double)));
  b->w64 = mixed ? nullptr : reinterpret_cast<double *>(take(3 * cap * sizeof(double)));
  b->q32 = mixed ? reinterpret_cast<float *>(take(P32_PLANES * cap * sizeof(float))) : nullptr;
  b->targets = take(cap * sizeof(Target<Fp64>));
  b->boxes = take(cap / kCellTile * sizeof(TileBox<double>));
  return o;
}

template <class V>
hipError_t run(const tsbts_ctx *c, const CellBufs &b, const int32_t *idx, int n_act, double eta,
               double *dtc, hipStream_t st) {
  using F = typename V::F;
  static_assert(sizeof(Target<V>) == sizeof(Target<Fp64>), "cell_layout");
  hipError_t e = launch_cell_sort(b.sort, c->p64, c->v64, sizeof(F) == 4, c->n, c->npad, idx,
                                  n_act, st);
  if (e != hipSuccess) return e;
  ScatterArgs a;
  a.s = b.sort;
  a.p64 = c->p64;
  a.v64 = c->v64;
  a.p32 = c->p32;
  a.npad = c->npad;
  a.n = c->n;
  a.idx = idx;
  a.n_act = n_act;
  a.q64 = b.q64;
  a.w64 = b.w64;
  a.q32 = b.q32;
  a.cap = c->npad;
  a.targets = b.targets;
  hipLaunchKernelGGL((k_cell_scatter<V>), dim3(static_cast<unsigned>((c->n + kWG - 1) / kWG)),
                     dim3(kWG), 0, st, a);
  CellArgs A;
  A.p32 = b.q32;
  A.p64 = b.q64;
  A.v64 = b.w64;
  A.npad = c->npad;
  A.n = c->n;
  A.n_tiles = static_cast<int>((c->n + kCellTile - 1) / kCellTile);
  A.origin = b.sort.origin;
  A.targets = b.targets;
  A.boxes = b.boxes;
  A.n_act = n_act;
  A.eps2 = c->eps * c->eps;
  A.eta = eta;
  A.dtc = dtc;
  constexpr int W = kWG / 64;  // waves of a workgroup
  hipLaunchKernelGGL((k_cell_boxes<V>), dim3((A.n_tiles + W - 1) / W), dim3(kWG), 0, st, A);
  hipLaunchKernelGGL((k_timestep_cells<V>), dim3((n_act + kGroup - 1) / kGroup), dim3(kWG), 0,
                     st, A, A.p32, A.p64, A.v64, static_cast<const Target<V> *>(b.targets),
                     static_cast<const TileBox<F> *>(b.boxes), dtc);
  return hipGetLastError();
}

}  // namespace

bool cells_criterion_applies(const tsbts_ctx *c, int64_t n_act) {
  // a call tuned to a kernel form keeps it
  if (c->tune_sym != 2 || c->tune_split != 2 || !automatic_form(c)) return false;
  // The order and the tests take as long as kPairs pairs and kTargets targets of the gather
  // kernels (half as many in float64 from kShareMaxAct targets).  Measured either side of
  // the line (us, this / gather): mixed N = 16384 k = 7061 72 / 71, 7300 70 / 78; 32768 4023
  // 79 / 74, 4280 79 / 87; 65536 2669 105 / 108, 2840 100 / 117; 131072 1992 153 / 157, 2120
  // 156 / 170; 262144 1500 238 / 214, 1661 241 / 248; 524288 1485 415 / 427, 1580 427 / 483;
  // 1048576 1100 786 / 635, 1391 763 / 774.  Float64 N = 8400 k = 6643 71 / 67, 7834 68 / 85;
  // 12000 4857 70 / 66, 5406 66 / 77; 18000 4351 71 / 84.
  constexpr int64_t kPairs = int64_t(90) << 20, kTargets = 1300;
  // Below kShareMaxAct targets the float64 gather kernels (waves share the targets) are
  // faster, and the line lies higher; for many particles it flattens.  Measured: N = 16384
  // k = 3953 67 / 59; 20011 3759 75 / 72, 4000 72 / 72; 32768 2600 83 / 78, 2804 83 / 85;
  // 65536 1700 109 / 103, 1892 108 / 114; 131072 1200 163 / 135, 1436 153 / 164; 262144 1000
  // 255 / 209, 1135 243 / 256; 524288 800 422 / 404, 900 420 / 441; 1048576 650 769 / 667, 850
  // 746 / 839.
  constexpr int64_t kPairs64 = 60000000, kTargets64 = 900;
  constexpr int64_t kMany = int64_t(1) << 19, kManyTargets64 = 860;
  const bool fp64 = c->precision == TSBTS_FP64;
  if (fp64 && n_act < kShareMaxAct)
    return n_act * c->n >= kPairs64 + kTargets64 * c->n ||
           (c->n >= kMany && n_act >= kManyTargets64);
  const int64_t pairs = n_act * c->n * (fp64 ? 2 : 1);
  return pairs >= kPairs + kTargets * c->n;
}

bool cells_prepare(tsbts_ctx *c, hipStream_t st) {
  if (c->cell_buf) return true;
  // the other kernels serve a captured call, and every call once the memory was refused
  if (c->cell_refused || !may_allocate(st)) return false;
  CellBufs b;
  if (hipMalloc(&c->cell_buf, cell_layout(c, nullptr, &b)) != hipSuccess) {
    (void)hipGetLastError();
    c->cell_buf = nullptr;
    c->cell_refused = true;
    return false;
  }
  return true;
}

hipError_t launch_timestep_cells(tsbts_ctx *c, const int32_t *idx, int n_act, double eta,
                                 double *dtc, hipStream_t st) {
  if (!c->cell_buf) return hipErrorNotReady;
  CellBufs b;
  cell_layout(c, static_cast<char *>(c->cell_buf), &b);
  if (c->precision == TSBTS_FP64) return run<Fp64>(c, b, idx, n_act, eta, dtc, st);
  if (c->flags & TSBTS_FLAG_HILO_SEPARATION)
    return run<MixHiLo>(c, b, idx, n_act, eta, dtc, st);
  return run<MixSep64>(c, b, idx, n_act, eta, dtc, st);
}

}  // namespace tsbts
