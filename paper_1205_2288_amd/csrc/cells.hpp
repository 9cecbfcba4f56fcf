// Spatial order of the predicted particles: a counting sort into cells of a grid whose
// planes are sample quantiles of each coordinate, numbered along a Morton curve, so that
// consecutive particles of the order are near each other whatever the density profile.
// The order serves kernels that treat tiles of kCellTile consecutive particles together;
// their results do not depend on which order that is.
//
// Five short launches: sampled planes (with the counters cleared), cell and rank of every
// particle (an integer atomic each, so particles of one cell come in no fixed order),
// the same for the targets, the scan of both counts, and the scatter, which belongs to
// the caller (it knows the planes it needs).  32768 cells: four particles each at 2^17.
#pragma once

#include "internal.hpp"

namespace tsbts {

constexpr int kCellBits = 5;                       // planes per coordinate: 2^5 - 1
constexpr int kCellSide = 1 << kCellBits;
constexpr int kCells = 1 << (3 * kCellBits);
constexpr int kCellSamples = 256;                  // sampled particles per coordinate
constexpr int kCellTile = 64;                      // particles per tile: one per lane

// Device arrays of one sort of n particles and k targets.
struct CellSort {
  double *origin;     // [6]: median of the sampled positions, mean of the sampled velocities
  float *planes;      // [3][kCellSide]: ascending planes about the origin, the last one +inf
  int32_t *count;     // [2][kCells]: particles, then targets; after the scan: first places
  int32_t *key;       // [n] cell of each particle
  int32_t *rank;      // [n] its rank in the cell
  int32_t *trank;     // [k] rank of each target in its cell
};

// Place of particle j, and of target q (particle g), in the two orders.
__device__ __forceinline__ int32_t cell_place(const CellSort &s, int64_t j) {
  return s.count[s.key[j]] + s.rank[j];
}
__device__ __forceinline__ int32_t cell_target_place(const CellSort &s, int q, int64_t g) {
  return s.count[kCells + s.key[g]] + s.trank[q];
}

// Everything but the scatter, for the positions p64[0..2][npad] and velocities
// v64[0..2][npad] (rounded to float32 where the caller's pairs see them so).
hipError_t launch_cell_sort(const CellSort &s, const double *p64, const double *v64,
                            bool v_float, int64_t n, int64_t npad, const int32_t *idx,
                            int n_act, hipStream_t st);

// Criterion over the spatial order (timestep_cells.hip): whether it serves a call of
// n_act targets; its buffers, host set-up made by every entry point that goes on to
// launch_timestep with such a call (false when they cannot be had, the other kernels then
// serve it); and its launch (hipErrorNotReady, with nothing launched, without the buffers).
bool cells_criterion_applies(const tsbts_ctx *c, int64_t n_act);
bool cells_prepare(tsbts_ctx *c, hipStream_t st);
hipError_t launch_timestep_cells(tsbts_ctx *c, const int32_t *idx, int n_act, double eta,
                                 double *dtc, hipStream_t st);

}  // namespace tsbts
