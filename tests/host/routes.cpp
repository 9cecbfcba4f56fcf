// The library's host-side rules (which kernel form, split, reduction and counter a call
// takes) behind a C interface, on a context that only has the fields the rules read.
#include <algorithm>

#include "cells.hpp"
#include "internal.hpp"

using namespace tsbts;

extern "C" {

tsbts_ctx *route_ctx(int64_t n, int precision) {
  tsbts_ctx *c = new tsbts_ctx();
  c->n = n;
  c->npad = round_up(n, kPad);
  c->precision = precision;
  // never read or written: the rules only compare and offset these
  c->part = reinterpret_cast<double *>(0x10000);
  c->done = reinterpret_cast<uint32_t *>(0x20000);
  return c;
}
void route_free(tsbts_ctx *c) { delete c; }

// Counter of a small-set force call with partials in the context's array or another, and of
// a small-set criterion call, as offsets.
int route_force_done(const tsbts_ctx *c, int own) {
  double *part = own ? c->part : c->part + 1;
  return static_cast<int>(force_done(c, part) - c->done);
}
int route_step_done(const tsbts_ctx *c) { return static_cast<int>(step_done(c) - c->done); }
int route_share_done(const tsbts_ctx *c, int which) {
  return static_cast<int>(share_done(c, which) - c->done);
}
int route_done_counts() { return kDoneCounts; }
int route_share_tiles() { return kShareTiles; }
}

extern "C" {
int64_t route_partials(const tsbts_ctx *c, int k) {
  const bool fused = k > kSmallAct && k < kShareMaxAct;
  return std::max(partial_elems_needed(c, k), fused ? fused_partials_needed(c, k) : 0);
}
int64_t route_reserve(const tsbts_ctx *c) {
  return std::max(gather_partials_reserve(c), share_partials_reserve(c));
}
}

extern "C" {
int route_force_rows(int slices, int64_t targets, int shared) {
  return force_rows_reduce(slices, targets, shared != 0) ? 1 : 0;
}
int route_step_rows(int slices, int64_t targets, int shared) {
  return step_rows_reduce(slices, targets, shared != 0) ? 1 : 0;
}
}

extern "C" int route_cells(const tsbts_ctx *c, int64_t k) {
  return cells_criterion_applies(c, k) ? 1 : 0;
}

extern "C" {
int route_apart(const tsbts_ctx *c, int k) { return criterion_apart(c, k) ? 1 : 0; }
}

extern "C" {
void route_tune_blocks(tsbts_ctx *c, int blocks) { c->tune_blocks = blocks; }
int route_share(const tsbts_ctx *c, int k) {
  return (share_force(c, k).chunk != 0) + 2 * (share_step(c, k).chunk != 0);
}
}

extern "C" int route_first(const tsbts_ctx *c, int k) { return criterion_first(c, k) ? 1 : 0; }

extern "C" int route_energy_bits(int64_t ntp) { return energy_part_bits(ntp); }
