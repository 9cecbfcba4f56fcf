"""Active sets whose targets the waves of a workgroup share (33 to 4095 targets): force and
potential against the oracle, the criterion bit for bit against the LDS-staged kernel, at
target counts around a wave, with units that pass the padding (a plane length that is not
a multiple of 1024), in each split of the sources, and next to the limits of the form."""
import numpy as np
import pytest

import oracle
from workloads import plummer
from gpu_util import rel_err, rel_err_vec, summary, make_ctx, TOL

pytestmark = pytest.mark.gpu

CASES = [("fp64", "f64"), ("mixed", "hilo"), ("mixed", "f64")]
# (particles, targets): one and several units, few and many slices, j-parts of 16, 64, 256
SHAPES = [(40, 33), (300, 64), (1500, 65), (9000, 257), (9000, 4095), (9000, 4096),
          (66000, 100), (66000, 513), (66000, 4095)]


@pytest.mark.parametrize("prec,sep", CASES)
@pytest.mark.parametrize("n,k", SHAPES)
def test_shared_targets(prec, sep, n, k):
    eps, eta = 1 / 256, 0.1
    r, v, m = plummer(n, 6100 + k, masses="loguniform")
    idx = np.random.default_rng(k).permutation(n)[:k].astype(np.int32)
    ctx = make_ctx(n, eps, prec, sep)
    ctx.bind(r, v, m)
    ctx.predict(0.0)
    acc, pot = (x.cpu().numpy() for x in ctx.force(idx, 0.0))
    bare = ctx.force(idx, 0.0, with_pot=False)[0].cpu().numpy()
    dtc = ctx.timestep(idx, eta).cpu().numpy()
    ctx.tune(ipl=1)
    assert np.array_equal(dtc, ctx.timestep(idx, eta).cpu().numpy())
    ctx.close()
    assert np.array_equal(acc, bare)
    s = np.arange(0, k, max(1, k // 200))
    ra, rp = oracle.force(r, m, eps, idx[s])
    e = summary(rel_err_vec(acc[:, s], ra))
    assert e["median"] <= TOL[prec]["median"] and e["max"] <= TOL[prec]["max"], e
    e = rel_err(pot[s], rp)
    assert e.max() <= TOL[prec]["max"], summary(e)
