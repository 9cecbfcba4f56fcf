"""The fused force + criterion of sets whose targets the waves of a workgroup share: the two
separate kernels' values bit for bit (the force's split, part of a unit past the padding,
one slice, few and many of them, each unit size; float32 sums are the same numbers too)."""
import numpy as np
import pytest
import torch

from workloads import plummer
from gpu_util import make_ctx

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,sep,newton", [("fp64", "f64", False), ("mixed", "f64", False),
                                             ("mixed", "hilo", False), ("mixed", "f64", True)])
@pytest.mark.parametrize("n,k", [(33, 33), (40, 34), (256, 64), (513, 513), (1000, 65),
                                 (2600, 129), (4097, 777), (9000, 4095), (30011, 3999)])
def test_shared_fused_equals_separate_kernels(prec, sep, newton, n, k):
    r, v, m = plummer(n, 8400 + n, masses="loguniform")
    ctx = make_ctx(n, 1 / 256, prec, sep, newton)
    ctx.bind(r, v, m)
    ctx.predict(0.0)
    idx = ctx.idx(np.random.default_rng(n).permutation(n)[:k].astype(np.int32))
    acc, pot, dtc = ctx.force_criterion(idx, 0.0, 0.1)
    alone = ctx.force_criterion(idx, 0.0, 0.1, with_pot=False)
    acc2, pot2 = ctx.force(idx, 0.0)
    dtc2 = ctx.timestep(idx, 0.1)
    ctx.close()
    assert torch.equal(acc, acc2) and torch.equal(pot, pot2) and torch.equal(dtc, dtc2)
    assert torch.equal(alone[0], acc2) and torch.equal(alone[2], dtc2)
