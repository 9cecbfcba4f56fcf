"""Adjoint of few rows: the shared-row kernels (float64, fewer than 2^25 target-particle
pairs) and the LDS kernels' column batches (mixed), at sets around a wave, padding inside a
unit, each split of the columns and both sides of the limit.  Against the oracle (float64
sums of the same terms: check_adjoint's bounds), against the tiles of 256 that a tuned
chunk selects, and added to what the outputs hold."""
import numpy as np
import pytest
import torch

import oracle
from workloads import plummer, gaussian
from gpu_util import check_adjoint, make_ctx

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,sep", [("fp64", "f64"), ("mixed", "f64"), ("mixed", "hilo")])
@pytest.mark.parametrize("with_gp", [False, True])
@pytest.mark.parametrize("n,k", [(2, 1), (40, 40), (300, 64), (300, 65), (1000, 1000),
                                 (1537, 700), (5000, 33), (9000, 3728), (9000, 3729)])
def test_few_row_adjoint(prec, sep, n, k, with_gp):
    r, _, m = plummer(n, 7500 + n, masses="loguniform")
    idx = np.random.default_rng(k).permutation(n)[:k].astype(np.int32)
    ga, gp = gaussian((3, k), 5), gaussian(k, 6) if with_gp else None
    ctx = make_ctx(n, 1 / 64, prec, sep)
    ctx.bind(r, np.zeros((3, n)), m)
    ctx.predict(0.0)
    got = []
    for chunk in (0, 256):
        ctx.tune(chunk=chunk)
        gr = torch.full((3, n), 0.5, dtype=torch.float64, device="cuda")
        gm = torch.full((n,), -0.25, dtype=torch.float64, device="cuda")
        ctx.force_backward(idx, 0.0, torch.tensor(ga, device="cuda"),
                           None if gp is None else torch.tensor(gp, device="cuda"), gr, gm)
        got.append((gr.cpu().numpy() - 0.5, gm.cpu().numpy() + 0.25))
    ctx.close()
    gz = np.zeros(k) if gp is None else gp
    sr, sm = oracle.force_backward_scale(r, m, 1 / 64, idx, ga, gz)
    # two float64 orders of the same terms, sqrt(n) roundings each; mixed: the same float32
    # sums, so float64 alone differs
    tol = 4 * np.sqrt(n) * 2.3e-16
    for a, b, s in zip(got[0], got[1], (sr, sm)):
        assert (np.abs(a - b) <= tol * (s + 1.0)).all()
    if n <= 2000:
        rr, rm = oracle.force_backward(r, m, 1 / 64, idx, ga, gz)
        check_adjoint(got[0][0], got[0][1], rr, rm, sr, sm, prec, f"{n} {k}")
