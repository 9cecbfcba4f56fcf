"""Gradients through runs whose states are kept in one buffer: the same bits whatever the
number of steps between checkpoints (one: nothing is recomputed; more than the run's), for
a second backward pass, and for inputs that are views."""
import numpy as np
import pytest
import torch

from workloads import plummer
from gpu_util import make_ctx
from paper_1205_2288_amd.autograd import tsbts_block_leapfrog, tsbts_leapfrog

pytestmark = pytest.mark.gpu
STEPS = 4


def _grads(kind, prec, n, era, view):
    r, v, m = plummer(n, 7400 + n, masses="loguniform")
    ctx = make_ctx(n, 1 / 64, prec)
    x = [torch.tensor(a, dtype=torch.float64, device="cuda") for a in (r, v, m)]
    if view:  # particle-major memory behind the planes
        x[0], x[1] = (a.t().contiguous().t() for a in x[:2])
    x = [a.requires_grad_(True) for a in x]
    h = 1 / 256
    if kind == "shared":
        out = tsbts_leapfrog(*x, ctx, h, STEPS, era)
    else:
        dt = h * 2.0 ** (np.arange(n) % 3)
        out = tsbts_block_leapfrog(*x, ctx, dt, STEPS * h, era)
    w = [torch.cos(torch.arange(3 * n, dtype=torch.float64, device="cuda") + c).view(3, n)
         for c in range(2)]
    first = torch.autograd.grad(out, x, w, retain_graph=True)
    again = torch.autograd.grad(out, x, w)
    ctx.close()
    assert all(torch.equal(a, b) for a, b in zip(first, again))
    return [a.detach().cpu().numpy() for a in (*out, *first)]


@pytest.mark.parametrize("kind", ["shared", "block"])
@pytest.mark.parametrize("prec,n", [("fp64", 65), ("mixed", 700)])
def test_checkpoint_spacing(kind, prec, n):
    ref = _grads(kind, prec, n, STEPS, False)
    assert all(np.isfinite(a).all() for a in ref)
    for era, view in ((1, False), (3, False), (STEPS + 5, False), (2, True)):
        assert all(np.array_equal(a, b) for a, b in zip(ref, _grads(kind, prec, n, era, view)))


@pytest.mark.parametrize("kind", ["shared", "block"])
def test_memory_left_by_others(kind):
    # buffers that come from the allocator with another tensor's NaNs in them
    ref = _grads(kind, "fp64", 300, 2, False)
    for _ in range(3):
        left = [torch.full((c * 300,), float("nan"), dtype=torch.float64, device="cuda")
                for c in (1, 3, 3, 3, 6, 9, 10, 11, 11, 11, 12, 33)]
        del left
        assert all(np.array_equal(a, b) for a, b in zip(ref, _grads(kind, "fp64", 300, 2, False)))
