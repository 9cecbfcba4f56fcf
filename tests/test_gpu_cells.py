"""Criterion of large active sets over the spatial order (tiles that cannot change a target's
maximum or minimum are left out): equal bit for bit to the gather kernels (maxima and
minima are exact), at the smallest calls it serves, with ragged particle, target and tile
counts, and on sets whose order or bounds degenerate: one point, a line, equal velocities,
massless particles, far outliers, a distant moving frame, values that are not finite."""
import numpy as np
import pytest
import torch

import oracle
from workloads import plummer
from gpu_util import rel_err, summary, make_ctx

pytestmark = pytest.mark.gpu

CASES = [("fp64", "hilo"), ("mixed", "hilo"), ("mixed", "f64")]
# (particles, targets): full and ragged tiles, groups of 16 targets and chunks of 64 tiles
SHAPES = [(32768, 4180), (32769, 4201), (40000, 39999), (33000, 33000), (131071, 2021)]


def _sphere(n, kind):
    r, v, m = plummer(n, 5200 + n % 97, masses="loguniform")
    g = np.random.default_rng(n)
    if kind == "point":           # everything in one cell, a few coincident particles
        r = 0.5 + 1e-9 * g.standard_normal((3, n))
        r[:, 1:4] = r[:, :1]
    elif kind == "line":
        r[1:] = 0.25
    elif kind == "drift":         # no relative velocity: the free-fall term alone
        v = np.tile(np.array([[0.3], [-0.7], [0.2]]), (1, n))
    elif kind == "far":           # far from the origin, at a high common speed
        r, v = r + 1e5, v - 300.0
    elif kind == "massless":
        m = m.copy()
        m[g.random(n) < 0.9] = 0.0
    elif kind == "outliers":      # escapers and a tight pair
        r = r.copy()
        r[:, ::1000] *= 1e6
        r[:, 5] = r[:, 6] + 1e-7
    elif kind == "nonfinite":
        r, v = r.copy(), v.copy()
        r[0, 17], v[1, 4000], r[2, 9000] = np.inf, np.nan, np.nan
    return r, v, m


def _check(n, k, prec, sep, kind, eps=1 / 1024):
    r, v, m = _sphere(n, kind)
    idx = np.random.default_rng(k).permutation(n)[:k].astype(np.int32)
    ctx = make_ctx(n, eps, prec, sep)
    ctx.bind(r, v, m)
    ctx.predict(0.0)
    got = ctx.timestep(idx, 0.1).cpu().numpy()
    again = ctx.timestep(idx, 0.1).cpu().numpy()
    ctx.tune(symmetric=0, split=0)
    ref = ctx.timestep(idx, 0.1).cpu().numpy()
    ctx.close()
    assert np.array_equal(got, ref, equal_nan=True), \
        (np.flatnonzero(got != ref)[:10], got[got != ref][:5], ref[got != ref][:5])
    assert np.array_equal(got, again, equal_nan=True)
    return r, v, m, idx, got


@pytest.mark.parametrize("prec,sep", CASES)
@pytest.mark.parametrize("n,k", SHAPES)
def test_cells_criterion_equals_gather(prec, sep, n, k):
    r, v, m, idx, got = _check(n, k, prec, sep, "plummer")
    s = np.arange(0, k, k // 64)
    e = rel_err(got[s], oracle.timestep(r, v, m, 1 / 1024, 0.1, idx[s]))
    assert e.max() <= (1e-12 if prec == "fp64" else 2e-6), summary(e)


@pytest.mark.parametrize("prec", ["mixed", "fp64"])
@pytest.mark.parametrize("kind", ["point", "line", "drift", "far", "massless", "outliers",
                                  "nonfinite"])
def test_cells_criterion_degenerate_sets(prec, kind):
    _check(33001, 5001, prec, "f64", kind, eps=0.0 if kind in ("massless", "outliers") else 1 / 64)


def test_cells_criterion_after_corrector_and_on_another_stream():
    # the corrector rewrites the targets' velocities; the call on a side stream uses only
    # that stream's buffers and order
    n, k, h = 40000, 20000, 1 / 1024
    r, v, m = plummer(n, 5300)
    idx = np.random.default_rng(1).permutation(n)[:k].astype(np.int32)
    ctx = make_ctx(n, 1 / 256, "mixed")
    ctx.bind(r, v, m, dt=np.full(n, h))
    idx = ctx.idx(idx)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        ctx.predict(h, stream=side)
        acc = ctx.force(idx, h, with_pot=False, stream=side)[0]
        ctx.correct(idx, h, acc, stream=side)
        got = ctx.timestep(idx, 0.1, stream=side)
        ctx.tune(symmetric=0, split=0)
        ref = ctx.timestep(idx, 0.1, stream=side)
    side.synchronize()
    assert torch.equal(got, ref)
    ctx.close()
