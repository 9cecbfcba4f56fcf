"""Adjoint of partial sets on both sides of 2^25 target-particle pairs, where the kernels
change (float64: shared rows below it, tiles of 256 above; mixed: four columns in flight,
two), against the oracle: its float64 sums and each element's rounding scale."""
import numpy as np
import pytest
import torch

import oracle
from workloads import plummer, gaussian
from gpu_util import check_adjoint, make_ctx

pytestmark = pytest.mark.gpu
_ref = {}


def _oracle(n, k):
    if (n, k) not in _ref:
        r, _, m = plummer(n, 7500 + n, masses="loguniform")
        idx = np.random.default_rng(k).permutation(n)[:k].astype(np.int32)
        ga, gp = gaussian((3, k), 5), gaussian(k, 6)
        _ref[n, k] = (r, m, idx, ga, gp, oracle.force_backward(r, m, 1 / 64, idx, ga, gp),
                      oracle.force_backward_scale(r, m, 1 / 64, idx, ga, gp))
    return _ref[n, k]


@pytest.mark.parametrize("prec,sep", [("fp64", "f64"), ("mixed", "f64"), ("mixed", "hilo")])
@pytest.mark.parametrize("n,k", [(5000, 33), (9000, 3728), (9000, 3729)])
def test_partial_adjoint_matches_oracle(prec, sep, n, k):
    r, m, idx, ga, gp, (rr, rm), (sr, sm) = _oracle(n, k)
    ctx = make_ctx(n, 1 / 64, prec, sep)
    ctx.bind(r, np.zeros((3, n)), m)
    ctx.predict(0.0)
    gr, gm = ctx.force_backward(idx, 0.0, torch.tensor(ga, device="cuda"),
                                torch.tensor(gp, device="cuda"))
    check_adjoint(gr.cpu().numpy(), gm.cpu().numpy(), rr, rm, sr, sm, prec, f"{n} {k}")
    ctx.close()
