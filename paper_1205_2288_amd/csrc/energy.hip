// Total energy E = K + W for the energy-error diagnostic (Section 3), in float64:
//   K =  1/2 sum_i m_i |v_i|^2,   W = -sum_{i<j} m_i m_j (|r_i - r_j|^2 + eps^2)^(-1/2).
// The upper triangle of 256x256 particle tiles (I <= J) is enumerated in row order and cut
// into at most kMaxEB contiguous ranges of tile pairs (of parts of them where they are
// few), one per workgroup: for each pair,
// target i = 256 I + lane in registers, the sources of tile J through wave-uniform (scalar)
// loads, and on diagonal tiles only j > i counts.  Each lane sums its pairs in range
// order, the workgroup reduces its lanes in a fixed order into one partial, and a single
// workgroup then adds the partials in a fixed order, so the result is bit-reproducible and
// the partials take at most 2 kMaxEB float64 values whatever N.  1/sqrt is the hardware
// float64 estimate refined by one Newton step, y (3 - s y^2) / 2, folded into the sum (the
// half at the end): 11 instructions and 60 issue cycles per wave of pairs, 16 of them
// the estimate.  Bound by vector ALU issue; sources staged in LDS (two broadcast reads of
// 16 bytes per pair, 64 of 68 cycles of a CU's LDS) were as slow as the arithmetic.
// N = 131072: 4.06 -> 3.60 ms.  (s from 5.6e-309, below which y^2 overflows: rsqrt_f64.)
#include <algorithm>

#include "internal.hpp"

namespace tsbts {
namespace {

constexpr int kTE = 256;
constexpr int64_t kMaxEB = 8192;  // workgroups (and partials) of the pair kernel
// With few tile pairs each is cut into parts of its sources, up to kMaxParts and about
// kPartItems items: a serial chain of 256 pairs per lane would set the time (us, whole
// tile pairs and parts: N = 1000 24.6, 7.6; 4096 25.0, 12.8; 8192 36.5, 27.0).  Two parts pay
// up to kPartItemsTwo items, whose last round of workgroups would be nearly empty otherwise
// (N = 16384 76.1, 71.6; 18077 88.5, 83.2; 9000 in 8 parts instead of 4 30.1, 31.6; 22000 in
// 2 instead of 1 117.1, 117.7).
constexpr int64_t kPartItems = 4096, kPartItemsTwo = 6144;
constexpr int kMaxPartBits = 3;
}  // namespace

int energy_part_bits(int64_t ntp) {
  int q = 0;
  while (q < kMaxPartBits && (2 * ntp << q) <= (q == 0 ? kPartItemsTwo : kPartItems)) ++q;
  return q;
}

namespace {

struct EnergyArgs {
  int64_t n;
  const double *r, *v, *m;
  double eps2;
  int64_t T;       // tile rows
  int64_t ntp;     // tile pairs T (T + 1) / 2
  int64_t nb;      // workgroups: min(ntp << part_bits, kMaxEB)
  double *part;    // [nb][2]
  double *out;
  int part_bits;  // log2 of the parts of each tile pair's sources
};

// Tile pair b -> (I, J), I <= J, rows enumerated I = 0, 1, ... with T - I pairs each.
__device__ __forceinline__ void tile_pair(int64_t b, int64_t T, int64_t &I, int64_t &J) {
  const double a = 2.0 * static_cast<double>(T) + 1.0;
  int64_t i = static_cast<int64_t>((a - sqrt(a * a - 8.0 * static_cast<double>(b))) * 0.5);
  auto first = [T](int64_t r) { return r * T - r * (r - 1) / 2; };
  while (i > 0 && first(i) > b) --i;
  while (first(i + 1) <= b) ++i;
  I = i;
  J = i + (b - first(i));
}

// Sum over sources [j0, j1) of m_j (3 - s y^2) y, twice m_j / sqrt(s), against one target;
// with MASK only over j > i.
template <int MASK>
__device__ __forceinline__ double energy_tile(const EnergyArgs &A, int64_t j0, int64_t j1,
                                              int64_t i, double xi, double yi, double zi) {
  const int64_t n = A.n;
  double w = 0.0;
#pragma unroll 8
  for (int64_t j = j0; j < j1; ++j) {
    const double dx = A.r[j] - xi, dy = A.r[n + j] - yi, dz = A.r[2 * n + j] - zi;
    double s = fma(dx, dx, fma(dy, dy, fma(dz, dz, A.eps2)));
    double m = A.m[j];
    if (MASK && j <= i) {
      s = 1.0;
      m = 0.0;
    }
    const double y = rsq_f64_approx(s);
    w = fma(m * y, fma(-s, y * y, 3.0), w);
  }
  return w;
}

__global__ __launch_bounds__(kWG) void k_energy_pairs(EnergyArgs A) {
  __shared__ double red[2][kWG / 64];
  const int tid = threadIdx.x;
  const int64_t n = A.n;
  // this workgroup's contiguous range of the parts of tile pairs
  const int64_t items = A.ntp << A.part_bits;
  const int64_t b0 = blockIdx.x * items / A.nb, b1 = (blockIdx.x + 1) * items / A.nb;
  const int len = kTE >> A.part_bits;
  double pw = 0.0, pk = 0.0;
  for (int64_t b = b0; b < b1; ++b) {
    int64_t I, J;
    tile_pair(b >> A.part_bits, A.T, I, J);
    const int part = static_cast<int>(b) & ((1 << A.part_bits) - 1);
    const int64_t i = I * kTE + tid;
    // targets past the last particle read its position and count for nothing: they lie in
    // the last tile row, whose one pair is diagonal and leaves out every j <= i, and have no
    // mass and no kinetic energy
    const int64_t ii = i < n ? i : n - 1;
    const double xi = A.r[ii], yi = A.r[n + ii], zi = A.r[2 * n + ii];
    const double mi = i < n ? A.m[ii] : 0.0;
    if (I == J && part == 0 && i < n) {
      const double vx = A.v[i], vy = A.v[n + i], vz = A.v[2 * n + i];
      pk += 0.5 * mi * (vx * vx + vy * vy + vz * vz);
    }
    const int64_t j0 = J * kTE + part * len, j1 = j0 + len < n ? j0 + len : n;
    const double w = I != J ? energy_tile<0>(A, j0, j1, i, xi, yi, zi)
                            : energy_tile<1>(A, j0, j1, i, xi, yi, zi);
    pw = fma(mi, 0.5 * w, pw);
  }
  pw = wave_sum(pw);
  pk = wave_sum(pk);
  if ((tid & 63) == 0) {
    red[0][tid >> 6] = pw;
    red[1][tid >> 6] = pk;
  }
  __syncthreads();
  if (tid == 0) {
    double sw = 0.0, sk = 0.0;
    for (int k = 0; k < kWG / 64; ++k) {
      sw += red[0][k];
      sk += red[1][k];
    }
    A.part[2 * blockIdx.x] = sw;
    A.part[2 * blockIdx.x + 1] = sk;
  }
}

constexpr int kRedWG = 1024;
__global__ __launch_bounds__(kRedWG) void k_energy_reduce(EnergyArgs A) {
  __shared__ double sw[kRedWG], sk[kRedWG];
  const int t = threadIdx.x;
  double w = 0.0, k = 0.0;
  for (int64_t b = t; b < A.nb; b += kRedWG) {
    w += A.part[2 * b];
    k += A.part[2 * b + 1];
  }
  sw[t] = w;
  sk[t] = k;
  __syncthreads();
  for (int s = kRedWG / 2; s > 0; s >>= 1) {
    if (t < s) {
      sw[t] += sw[t + s];
      sk[t] += sk[t + s];
    }
    __syncthreads();
  }
  if (t == 0) {
    A.out[0] = sk[0];
    A.out[1] = -sw[0];
  }
}

}  // namespace

int64_t energy_partials_needed(const tsbts_ctx *c) {
  const int64_t T = (c->n + kTE - 1) / kTE;
  const int64_t ntp = T * (T + 1) / 2;
  return 2 * std::min<int64_t>(ntp << energy_part_bits(ntp), kMaxEB);  // two per workgroup
}

hipError_t launch_energy(tsbts_ctx *c, const double *r, const double *v, const double *m,
                         double *out, hipStream_t st) {
  EnergyArgs A;
  A.n = c->n;
  A.r = r;
  A.v = v;
  A.m = m;
  A.eps2 = c->eps * c->eps;
  A.T = (c->n + kTE - 1) / kTE;
  A.ntp = A.T * (A.T + 1) / 2;
  A.part_bits = energy_part_bits(A.ntp);
  A.nb = std::min<int64_t>(A.ntp << A.part_bits, kMaxEB);
  A.part = c->epart;
  A.out = out;
  hipLaunchKernelGGL(k_energy_pairs, dim3(static_cast<unsigned>(A.nb)), dim3(kWG), 0, st, A);
  hipLaunchKernelGGL(k_energy_reduce, dim3(1), dim3(kRedWG), 0, st, A);
  return hipGetLastError();
}

}  // namespace tsbts
