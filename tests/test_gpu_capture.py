"""A context's first criterion call captured, from the sizes where an uncaptured one would
allocate: the spatial order's, the symmetric kernels' and a split call's buffers.  The
capture completes, and every replay gives the eager call's values bit for bit."""
import numpy as np
import pytest
import torch

from workloads import plummer
from gpu_util import make_ctx
from paper_1205_2288_amd import _lib as L

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,n,k,split", [("mixed", 33000, 33000, 2), ("fp64", 33000, 33000, 2),
                                            ("mixed", 40000, 20000, 2), ("fp64", 40000, 20000, 2),
                                            ("mixed", 50000, 42240, 1), ("fp64", 12000, 9000, 1)])
def test_first_criterion_in_a_capture(prec, n, k, split):
    r, v, m = plummer(n, 7800 + n, masses="loguniform")
    ctx = make_ctx(n, 1 / 256, prec)
    ctx.tune(split=split)
    ctx.bind(r, v, m)
    ctx.predict(0.0)
    idx = ctx.idx(np.random.default_rng(n).permutation(n)[:k].astype(np.int32))
    d = torch.zeros(k, dtype=torch.float64, device="cuda")
    stream, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=stream):
        L.tsbts_timestep(ctx.ctx, idx, 0.1, d)
    for _ in range(3):
        d.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(d, ctx.timestep(idx, 0.1))
    ctx.close()
