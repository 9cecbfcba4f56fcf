"""A force call on the fixed array of partials beside the same context's own force and
criterion calls on another stream (neither waits for the other): the values of the calls
made one after the other, bit for bit."""
import numpy as np
import pytest
import torch

from workloads import plummer
from gpu_util import make_ctx
from paper_1205_2288_amd import _lib as L

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,n,k", [("mixed", 5000, 9), ("fp64", 16000, 3),
                                      ("mixed", 2000, 100)])
def test_fixed_array_calls_beside_the_contexts(prec, n, k):
    r, v, m = plummer(n, 8100 + n, masses="loguniform")
    ctx = make_ctx(n, 1 / 256, prec)
    ctx.bind(r, v, m)
    ctx.predict(0.0)
    g = np.random.default_rng(n)
    a_idx, b_idx = (ctx.idx(g.permutation(n)[:k].astype(np.int32)) for _ in range(2))
    new = lambda *s: torch.zeros(s, dtype=torch.float64, device="cuda")  # noqa: E731
    want_a, want_b, want_d = new(3, k), new(3, k), new(k)
    L.tsbts_force(ctx.ctx, a_idx, 0.0, want_a)
    L.tsbts_force_noalloc(ctx.ctx, b_idx, 0.0, want_b)
    L.tsbts_timestep(ctx.ctx, a_idx, 0.1, want_d)
    torch.cuda.synchronize()
    reps = 50
    a, b, d = new(reps, 3, k), new(reps, 3, k), new(reps, k)
    one, two = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    for i in range(reps):
        L.tsbts_force(ctx.ctx, a_idx, 0.0, a[i], None, one)
        L.tsbts_force_noalloc(ctx.ctx, b_idx, 0.0, b[i], None, two)
        L.tsbts_timestep(ctx.ctx, a_idx, 0.1, d[i], one)
    torch.cuda.synchronize()
    ctx.close()
    assert torch.equal(a, want_a.expand_as(a))
    assert torch.equal(b, want_b.expand_as(b))
    assert torch.equal(d, want_d.expand_as(d))
