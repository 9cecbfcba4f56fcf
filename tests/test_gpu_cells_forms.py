"""The spatial order's criterion launched by itself, so that it and no other form serves the
call: equal bit for bit to the gather kernels below the sizes that it is chosen for (fewer
particles than a tile or than samples, fewer targets than a group, ragged groups) and above
131072 particles, where a call that takes it is checked too."""
import ctypes

import numpy as np
import pytest
import torch

from workloads import plummer
from gpu_util import make_ctx
from paper_1205_2288_amd import _lib as L

pytestmark = pytest.mark.gpu
PREPARE = "_ZN5tsbts13cells_prepareEP9tsbts_ctxP12ihipStream_t"
LAUNCH = "_ZN5tsbts21launch_timestep_cellsEP9tsbts_ctxPKiidPdP12ihipStream_t"
APPLIES = "_ZN5tsbts23cells_criterion_appliesEPK9tsbts_ctxl"
P, D = ctypes.c_void_p, ctypes.c_double


def _fn(name, res, *args):
    f = getattr(L.lib, name)
    f.restype, f.argtypes = res, list(args)
    return f


def launch_cells(ctx, idx, eta, out):
    """hipError_t of the form's own launch (600: its buffers are not there)."""
    f = _fn(LAUNCH, ctypes.c_int, P, P, ctypes.c_int, D, P, P)
    return f(ctx.ctx, idx.data_ptr(), idx.numel(), eta, out.data_ptr(),
             torch.cuda.current_stream().cuda_stream)


def applies(ctx, k):
    return _fn(APPLIES, ctypes.c_bool, P, ctypes.c_int64)(ctx.ctx, k)


def _ctx(n, prec, sep="f64"):
    r, v, m = plummer(n, 8300 + n % 89, masses="loguniform")
    ctx = make_ctx(n, 1 / 256, prec, sep)
    ctx.bind(r, v, m)
    ctx.predict(0.0)
    return ctx


@pytest.mark.parametrize("prec,sep", [("fp64", "f64"), ("mixed", "f64"), ("mixed", "hilo")])
@pytest.mark.parametrize("n,k", [(1, 1), (2, 1), (17, 17), (63, 15), (64, 16), (65, 17),
                                 (200, 33), (513, 500), (4097, 100)])
def test_form_on_small_sets(prec, sep, n, k):
    ctx = _ctx(n, prec, sep)
    idx = ctx.idx(np.random.default_rng(n).permutation(n)[:k].astype(np.int32))
    assert _fn(PREPARE, ctypes.c_bool, P, P)(ctx.ctx, None)
    got = torch.zeros(k, dtype=torch.float64, device="cuda")
    assert launch_cells(ctx, idx, 0.1, got) == 0
    assert not applies(ctx, k)
    assert torch.equal(got, ctx.timestep(idx, 0.1))
    ctx.close()


@pytest.mark.parametrize("prec,n,k", [("mixed", 262144, 1701), ("fp64", 200003, 1300)])
def test_call_above_the_benchmark_size(prec, n, k):
    ctx = _ctx(n, prec)
    idx = ctx.idx(np.random.default_rng(n).permutation(n)[:k].astype(np.int32))
    assert applies(ctx, k)
    got = ctx.timestep(idx, 0.1)
    again = torch.zeros_like(got)
    assert launch_cells(ctx, idx, 0.1, again) == 0  # the call left the form's buffers
    ctx.tune(symmetric=0, split=0)
    assert not applies(ctx, k)
    ref = ctx.timestep(idx, 0.1)
    ctx.close()
    assert torch.equal(got, ref) and torch.equal(again, ref)


@pytest.mark.parametrize("prec,n,k", [("mixed", 131072, 3500), ("fp64", 131072, 2500)])
def test_combined_call_as_a_contexts_first(prec, n, k):
    # nothing else has allocated the form's buffers, and the call takes it all the same
    ctx = _ctx(n, prec)
    idx = ctx.idx(np.random.default_rng(n).permutation(n)[:k].astype(np.int32))
    assert applies(ctx, k)
    got = ctx.force_criterion(idx, 0.0, 0.1, with_pot=False)[2]
    again = torch.zeros_like(got)
    assert launch_cells(ctx, idx, 0.1, again) == 0
    ctx.close()
    assert torch.equal(got, again)
