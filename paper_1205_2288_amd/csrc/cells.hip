// Counting sort of the predicted particles into spatial cells (cells.hpp).
#include "cells.hpp"

namespace tsbts {
namespace {

constexpr int kScanWG = 1024;

// Block 0: the planes, every (kCellSamples / kCellSide)-th of the sorted samples of each
// coordinate (bitonic sort in LDS, one comparator per thread, the coordinates side by
// side), about their median, so that a set far from the origin of coordinates is ordered
// like one around it; and the mean sampled velocity.  The other blocks clear the counters.
// Bound by the latency of block 0's 36 barriers, about 5 us.
__global__ __launch_bounds__(3 * kCellSamples / 2) void k_cell_planes(CellSort s,
                                                                      const double *p64,
                                                                      const double *v64,
                                                                      int v_float, int64_t n,
                                                                      int64_t npad) {
  constexpr int H = kCellSamples / 2;
  static_assert(H == 128, "two waves per coordinate");
  const int t = threadIdx.x;
  if (blockIdx.x > 0) {
    const int e = (blockIdx.x - 1) * 3 * H + t;
    if (e < 2 * kCells) s.count[e] = 0;
    return;
  }
  __shared__ double x[3][kCellSamples];
  __shared__ double vs[6];
  const int c = t / H, i = t - c * H;
  double vel = 0.0;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int e = 2 * i + h;
    const int64_t j = e * n / kCellSamples;
    x[c][e] = p64[c * npad + j];
    double v = v64[c * npad + j];
    if (v_float) v = static_cast<float>(v);
    vel += fabs(v) < __builtin_inf() ? v : 0.0;  // (any finite reference will do)
  }
  vel = wave_sum(vel);
  if ((t & 63) == 0) vs[t >> 6] = vel;
  __syncthreads();
  for (int size = 2; size <= kCellSamples; size <<= 1) {
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      const int a = 2 * i - (i & (stride - 1)), b = a + stride;
      const double u = x[c][a], v = x[c][b];
      const bool up = (a & size) == 0;
      if ((u > v) == up) {
        x[c][a] = v;
        x[c][b] = u;
      }
      __syncthreads();
    }
  }
  const double mid = x[c][H];
  if (i < kCellSide)
    s.planes[c * kCellSide + i] =
        i + 1 < kCellSide
            ? static_cast<float>(x[c][(i + 1) * (kCellSamples / kCellSide)] - mid)
            : __builtin_inff();
  if (i == 0) {
    s.origin[c] = mid;
    s.origin[3 + c] = (vs[2 * c] + vs[2 * c + 1]) / kCellSamples;
  }
}

__device__ __forceinline__ int spread3(int b) {  // bit i to bit 3 i
  int r = 0;
#pragma unroll
  for (int i = 0; i < kCellBits; ++i) r |= ((b >> i) & 1) << (3 * i);
  return r;
}

// Cell of every particle and its rank there.
__global__ __launch_bounds__(kWG) void k_cell_count(CellSort s, const double *p64, int64_t n,
                                                    int64_t npad) {
  __shared__ float pl[3 * kCellSide];
  if (threadIdx.x < 3 * kCellSide) pl[threadIdx.x] = s.planes[threadIdx.x];
  __syncthreads();
  const int64_t j = static_cast<int64_t>(blockIdx.x) * kWG + threadIdx.x;
  if (j >= n) return;
  int key = 0;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const float x = static_cast<float>(p64[c * npad + j] - s.origin[c]);
    int b = 0;  // planes at or below x, by binary search
#pragma unroll
    for (int h = kCellSide >> 1; h > 0; h >>= 1) b += pl[c * kCellSide + b + h - 1] <= x ? h : 0;
    key |= spread3(b) << c;
  }
  s.key[j] = key;
  s.rank[j] = atomicAdd(&s.count[key], 1);
}

__global__ __launch_bounds__(kWG) void k_cell_count_targets(CellSort s, const int32_t *idx,
                                                            int n_act) {
  const int q = blockIdx.x * kWG + threadIdx.x;
  if (q >= n_act) return;
  s.trank[q] = atomicAdd(&s.count[kCells + s.key[idx[q]]], 1);
}

// Exclusive scan in place of the particles' counts (block 0) and the targets' (block 1):
// kCells / kScanWG consecutive counts per thread, its sum scanned over the wave and the
// waves' sums over the block.
__global__ __launch_bounds__(kScanWG) void k_cell_scan(CellSort s) {
  constexpr int PER = kCells / kScanWG;
  static_assert(PER % 4 == 0, "whole int4 loads");
  __shared__ int32_t wsum[kScanWG / 64];
  int4 *x = reinterpret_cast<int4 *>(s.count + blockIdx.x * kCells) + threadIdx.x * (PER / 4);
  int4 y[PER / 4];
  int32_t sum = 0;
#pragma unroll
  for (int e = 0; e < PER / 4; ++e) {
    y[e] = x[e];
    sum += y[e].x + y[e].y + y[e].z + y[e].w;
  }
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  int32_t inc = sum;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int32_t up = __shfl_up(inc, o, 64);
    if (lane >= o) inc += up;
  }
  if (lane == 63) wsum[w] = inc;
  __syncthreads();
  int32_t at = inc - sum;
  for (int v = 0; v < w; ++v) at += wsum[v];
#pragma unroll
  for (int e = 0; e < PER / 4; ++e) {
    const int4 z = y[e];
    int4 o;
    o.x = at;
    o.y = o.x + z.x;
    o.z = o.y + z.y;
    o.w = o.z + z.z;
    at = o.w + z.w;
    x[e] = o;
  }
}

}  // namespace

hipError_t launch_cell_sort(const CellSort &s, const double *p64, const double *v64,
                            bool v_float, int64_t n, int64_t npad, const int32_t *idx,
                            int n_act, hipStream_t st) {
  constexpr int T = 3 * kCellSamples / 2;
  hipLaunchKernelGGL(k_cell_planes, dim3(1 + (2 * kCells + T - 1) / T), dim3(T), 0, st, s, p64,
                     v64, v_float ? 1 : 0, n, npad);
  hipLaunchKernelGGL(k_cell_count, dim3(static_cast<unsigned>((n + kWG - 1) / kWG)), dim3(kWG),
                     0, st, s, p64, n, npad);
  hipLaunchKernelGGL(k_cell_count_targets, dim3((n_act + kWG - 1) / kWG), dim3(kWG), 0, st, s,
                     idx, n_act);
  hipLaunchKernelGGL(k_cell_scan, dim3(2), dim3(kScanWG), 0, st, s);
  return hipGetLastError();
}

}  // namespace tsbts
