"""Few particles: the launches that finish their own reduction and those of one workgroup.

* block steps of up to 32 targets whose launch is a single workgroup (at most 256
  particles, padding tiles left out) against the separate predictor, force and criterion
  launches: the same run bit for bit, at particle counts around one and two tiles;
* sets of 33 targets and more whose partials the last workgroup of each 64 targets adds
  (at most 8 slices): force against the oracle, force and criterion unchanged over calls
  (the workgroup counts return to zero) and in a captured graph's replays."""
import numpy as np
import pytest
import torch

import oracle
from workloads import plummer
from gpu_util import rel_err_vec, summary, make_ctx, TOL
from paper_1205_2288_amd import _lib as L

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("n", [40, 255, 256, 257, 513])
def test_one_workgroup_block_steps(prec, n):
    from paper_1205_2288_amd.driver import NativeTSBTS
    r, v, m = plummer(n, 7200 + n, masses="loguniform")
    out = []
    for pol in (False, True):
        sim = NativeTSBTS(r, v, m, 1 / 64, eta=0.1, passes=2, era=1 / 16, dt_max=1 / 64,
                          precision=prec, predict_on_load=pol)
        sim.run(1 / 8)
        out.append((sim.stats["block_steps"], sim.stats["interactions"],
                    sim.ctx.r.cpu().numpy().copy(), sim.ctx.v.cpu().numpy().copy()))
        sim.close()
    assert out[0][:2] == out[1][:2]
    assert np.array_equal(out[0][2], out[1][2]) and np.array_equal(out[0][3], out[1][3])


@pytest.mark.parametrize("prec,sep", [("fp64", "f64"), ("mixed", "f64"), ("mixed", "hilo")])
@pytest.mark.parametrize("n,k", [(40, 33), (256, 64), (500, 65), (513, 513), (2000, 129)])
def test_tile_reductions(prec, sep, n, k):
    r, v, m = plummer(n, 7300 + n, masses="loguniform")
    idx = np.random.default_rng(n).permutation(n)[:k].astype(np.int32)
    ctx = make_ctx(n, 1 / 256, prec, sep)
    ctx.bind(r, v, m)
    ctx.predict(0.0)
    acc = ctx.force(idx, 0.0)[0].cpu().numpy()
    dtc = ctx.timestep(idx, 0.1).cpu().numpy()
    e = summary(rel_err_vec(acc, oracle.force(r, m, 1 / 256, idx)[0]))
    assert e["median"] <= TOL[prec]["median"] and e["max"] <= TOL[prec]["max"], e
    d_idx = ctx.idx(idx)
    a = torch.zeros((3, k), dtype=torch.float64, device="cuda")
    d = torch.zeros(k, dtype=torch.float64, device="cuda")
    stream = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=stream):
        for _ in range(2):
            L.tsbts_force(ctx.ctx, d_idx, 0.0, a, None)
            L.tsbts_timestep(ctx.ctx, d_idx, 0.1, d)
    for _ in range(3):
        a.zero_()
        d.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(a.cpu().numpy(), acc) and np.array_equal(d.cpu().numpy(), dtc)
        assert np.array_equal(ctx.force(idx, 0.0)[0].cpu().numpy(), acc)
    ctx.close()


@pytest.mark.parametrize("prec,n,k", [("fp64", 4000, 1984), ("mixed", 4000, 1984),
                                      ("fp64", 3000, 1500), ("fp64", 16384, 16384),
                                      ("mixed", 16384, 9000)])
def test_first_call_in_a_capture(prec, n, k):
    # a context's first force, criterion and adjoint on a set, captured: the scratch was
    # reserved, and what would allocate (the criterion's spatial order) is not taken
    r, v, m = plummer(n, 7600 + n, masses="loguniform")
    ctx = make_ctx(n, 1 / 256, prec)
    ctx.bind(r, v, m)
    ctx.predict(0.0)
    idx = ctx.idx(np.random.default_rng(n).permutation(n)[:k].astype(np.int32))
    new = lambda *s: torch.zeros(s, dtype=torch.float64, device="cuda")  # noqa: E731
    a, d, gr, gm = new(3, k), new(k), new(3, n), new(n)
    g = torch.cos(torch.arange(3 * k, dtype=torch.float64, device="cuda")).view(3, k)
    stream, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=stream):
        L.tsbts_force(ctx.ctx, idx, 0.0, a, None)
        L.tsbts_timestep(ctx.ctx, idx, 0.1, d)
        L.tsbts_force_backward(ctx.ctx, n, idx, 0.0, g, None, gr, gm)
    for _ in range(3):
        for x in (a, d, gr, gm):
            x.zero_()
        graph.replay()
        torch.cuda.synchronize()
        acc = ctx.force(idx, 0.0, with_pot=False)[0]
        wr, wm = ctx.force_backward(idx, 0.0, g, None)
        assert torch.equal(a, acc) and torch.equal(d, ctx.timestep(idx, 0.1))
        assert torch.equal(gr, wr) and torch.equal(gm, wm)
    ctx.close()


@pytest.mark.parametrize("n", [1, 31, 33, 255, 257, 700, 2000, 5633, 7936, 11500])
def test_energy_of_few_tiles(n):
    # each split of the tile pairs (8, 4, 2 and 1 parts), tails inside a part; float64 sums
    # of n (n - 1) / 2 terms of one sign: 1e-13 relative leaves sqrt(n^2) roundings ample room
    r, v, m = plummer(n, 7700 + n, masses="loguniform")
    ctx = make_ctx(n, 1 / 64, "fp64")
    ctx.bind(r, v, m)
    kin, pot = ctx.energy().cpu().numpy()
    ctx.close()
    phi = oracle.force(r, m, 1 / 64, np.arange(n, dtype=np.int32))[1]
    assert kin == pytest.approx(0.5 * (m * (v * v).sum(0)).sum(), rel=1e-13)
    assert pot == pytest.approx(0.5 * (m * phi).sum(), rel=1e-13)
