// The float64 reciprocal powers of a pair, alone in a kernel, for a count of operations.
#include "internal.hpp"

using namespace tsbts;

template <int POT>
__device__ void one(const double *in, double *out) {
  double pot = in[2];
  out[0] = scaled_inv_cube_f64<POT>(in[0], in[1], pot);
  out[1] = pot;
}
extern "C" __global__ void k_force_only(const double *in, double *out) { one<0>(in, out); }
extern "C" __global__ void k_with_potential(const double *in, double *out) { one<1>(in, out); }
