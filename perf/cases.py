"""The calls whose speed counts, from the smallest block step to the largest sums.

A program that uses this package integrates a star cluster: most of its calls are block
steps (predict all particles, force on the active ones, corrector, time-step criterion)
with anything from one to all particles active, driven one by one or by the native
scheduler; it measures the total energy now and then; and where it differentiates, it
calls the force adjoint, alone or inside a leapfrog run.  The particle sets are Plummer
spheres in Henon units, the softening and the mass spectra those of the repository's
workloads (256 to 131072 particles).

Every case names its kind; ``prepare`` builds the context and the inputs, ``run`` makes
one pass through the public entry points, ``exact`` evaluates the same sums in float64
with plain torch.
"""
import math

import numpy as np
import torch

from paper_1205_2288_amd import Context
from paper_1205_2288_amd.autograd import tsbts_block_leapfrog, tsbts_leapfrog
from paper_1205_2288_amd.driver import NativeTSBTS

ETA = 0.1
H0 = 2.0 ** -10  # smallest step of the block-step states


def listed():
    return [
        # the commonest call of a small run: a dozen particles due, everything latency
        dict(name="step_4k_13", kind="step", n=4096, k=13, eps=1 / 256, prec="mixed"),
        # one particle due in a mid-sized cluster, with the potential (diagnostics)
        dict(name="force_32k_1", kind="force", n=32768, k=1, eps=1 / 1024, prec="mixed"),
        # an ordinary block step: a few per cent of the particles, ragged sizes
        dict(name="step_30k_777", kind="step", n=30011, k=777, eps=1 / 1024, prec="mixed"),
        # the same kind of step in the float64 mode
        dict(name="step_20k_3000_fp64", kind="step", n=20011, k=3000, eps=1 / 256, prec="fp64"),
        # a large block step of the largest workload
        dict(name="step_131k_40k", kind="step", n=131072, k=40000, eps=1 / 4096, prec="mixed"),
        # a synchronising block step with the potential: every particle a target
        dict(name="force_131k_all", kind="force", n=131072, k=131072, eps=1 / 4096,
             prec="mixed"),
        # the energy diagnostic at era ends
        dict(name="energy_131k", kind="energy", n=131072, eps=1 / 4096, prec="mixed"),
        # force adjoint, all particles (the largest call of the benchmark step)
        dict(name="adjoint_131k_all", kind="adjoint", n=131072, k=131072, eps=1 / 4096,
             prec="mixed", pot=False),
        # gradients through a shared-step leapfrog: forward, recompute, backward
        dict(name="leapfrog_grad_8k", kind="leapfrog", n=8192, steps=16, era=8, eps=1 / 256,
             prec="mixed"),
        # gradients through a block schedule (three step levels, partial active sets)
        dict(name="block_grad_3k_fp64", kind="blocks", n=3001, levels=3, eps=1 / 256,
             prec="fp64"),
        # one era (three passes) of a whole native integration, small and mid-sized
        dict(name="era_256_fp64", kind="era", n=256, eps=1 / 64, era=1 / 8, prec="fp64"),
        dict(name="era_4k", kind="era", n=4096, eps=1 / 256, era=0.0, prec="mixed"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "force", "force", "energy", "adjoint",
                       "leapfrog", "blocks", "era"])
    prec = rng.choice(["mixed", "mixed", "fp64"])
    eps = 2.0 ** -rng.randint(6, 12)
    # float64 sums take about twice the time of mixed ones: three quarters of the particles
    top = 131072 if prec == "mixed" else 90000
    if kind in ("step", "force"):
        n = _log_int(rng, 256, top)
        k = n if rng.random() < 0.2 else _log_int(rng, 1, n)
        return dict(kind=kind, n=n, k=k, eps=eps, prec=prec)
    if kind == "energy":
        return dict(kind=kind, n=_log_int(rng, 1000, 131072), eps=eps, prec=prec)
    if kind == "adjoint":
        n = _log_int(rng, 500, top)
        k = n if rng.random() < 0.5 else _log_int(rng, 8, n // 2)
        return dict(kind=kind, n=n, k=k, eps=eps, prec=prec, pot=rng.random() < 0.5)
    if kind == "leapfrog":
        return dict(kind=kind, n=_log_int(rng, 500, 12000), steps=rng.randint(4, 16),
                    era=rng.choice([4, 8]), eps=eps, prec=prec)
    if kind == "blocks":
        return dict(kind=kind, n=_log_int(rng, 500, 8000), levels=rng.choice([2, 3]),
                    eps=eps, prec=prec)
    n = _log_int(rng, 128, 4096)
    # (fixed eras of two largest steps only where an era stays short)
    return dict(kind="era", n=n, eps=1 / 64 if n < 512 else 1 / 256,
                era=rng.choice([0.0, 1 / 32]) if n < 1500 else 0.0, prec=prec)


# ------------------------------------------------------------------ inputs
def _isotropic(g, mag):
    z = (1.0 - 2.0 * g.random(mag.size)) * mag
    phi = 2.0 * math.pi * g.random(mag.size)
    rho = np.sqrt(np.maximum(mag * mag - z * z, 0.0))
    return np.stack([rho * np.cos(phi), rho * np.sin(phi), z])


def _sphere(n, seed):
    """Plummer sphere, total mass 1, energy -1/4: positions, velocities [3, n], masses."""
    g = np.random.default_rng(seed)
    rad = np.empty(0)
    while rad.size < n:
        with np.errstate(divide="ignore"):
            x = 1.0 / np.sqrt(g.random(n + 16) ** (-2.0 / 3.0) - 1.0)
        rad = np.concatenate([rad, x[x < 10.0]])
    rad = rad[:n]
    q = np.empty(0)
    while q.size < n:
        x, y = g.random(2 * n + 64), g.random(2 * n + 64)
        q = np.concatenate([q, x[0.1 * y < x * x * (1.0 - x * x) ** 3.5]])
    vel = _isotropic(g, q[:n] * math.sqrt(2.0) * (1.0 + rad * rad) ** -0.25)
    pos = _isotropic(g, rad)
    m = 10.0 ** g.random(n)
    m /= m.sum()
    pos *= 3.0 * math.pi / 16.0
    vel *= math.sqrt(16.0 / (3.0 * math.pi))
    pos -= (pos * m).sum(axis=1, keepdims=True)
    vel -= (vel * m).sum(axis=1, keepdims=True)
    return pos, vel, m


def _targets(n, k, seed):
    g = np.random.default_rng(seed + 1)
    return np.sort(g.permutation(n)[:k]).astype(np.int32)


def _inputs(case, seed):
    """Host arrays of a case, from the seed alone."""
    n, kind = case["n"], case["kind"]
    r, v, m = _sphere(n, seed)
    g = np.random.default_rng(seed + 2)
    d = dict(r=r, v=v, m=m)
    if "k" in case:
        d["idx"] = _targets(n, case["k"], seed)
    if kind == "step":
        # the accelerations a cluster of this size has, and particles last stepped up to
        # eight smallest steps ago; all of the active ones are due at the block time
        rad = np.sqrt((r * r).sum(axis=0))
        d["a"] = -r * (rad * rad + 0.35) ** -1.5 + 0.05 * g.standard_normal((3, n))
        d["tb"] = 8 * H0
        d["t_last"] = d["tb"] - H0 * 2.0 ** g.integers(0, 4, n)
        d["dt"] = np.full(n, 64 * H0)
        d["dt"][d["idx"]] = d["tb"] - d["t_last"][d["idx"]]
    if kind == "adjoint":
        d["ga"] = g.standard_normal((3, case["k"]))
        d["gp"] = g.standard_normal(case["k"]) if case["pot"] else None
    if kind in ("leapfrog", "blocks"):
        d["wr"], d["wv"] = g.standard_normal((3, n)), g.standard_normal((3, n))
        d["h"] = 1 / 256
    if kind == "blocks":
        lev = g.integers(0, case["levels"], n)
        lev[:2] = 0, case["levels"] - 1
        d["dt"] = d["h"] * 2.0 ** lev
        d["t_end"] = d["h"] * 2 ** (case["levels"] - 1)
    return d


def _gpu(x):
    return None if x is None else torch.as_tensor(x, dtype=torch.float64, device="cuda")


def prepare(case, seed):
    kind, n = case["kind"], case["n"]
    d = _inputs(case, seed)
    s = dict(case=case)
    if kind == "era":
        s["sim"] = NativeTSBTS(d["r"], d["v"], d["m"], case["eps"], eta=ETA, passes=3,
                               dt_max=1 / 64, era=case["era"] or None, precision=case["prec"])
        s["sim"].era_step()  # the first era still starts from one common time
        s["start"] = s["sim"].checkpoint()
        return s
    ctx = s["ctx"] = Context(n, case["eps"], precision=case["prec"])
    if kind in ("leapfrog", "blocks"):
        for key in ("r", "v", "m"):
            s[key] = _gpu(d[key]).requires_grad_(True)
        s["wr"], s["wv"] = _gpu(d["wr"]), _gpu(d["wv"])
        s.update({key: d[key] for key in ("h", "dt", "t_end") if key in d})
        return s
    ctx.bind(d["r"], d["v"], d["m"], a=d.get("a"), t_last=d.get("t_last"), dt=d.get("dt"))
    if kind == "energy":
        return s
    s["idx"] = ctx.idx(d["idx"])
    s["tb"] = d.get("tb", 0.0)
    if kind == "adjoint":
        s["ga"], s["gp"] = _gpu(d["ga"]), _gpu(d["gp"])
        ctx.predict(0.0)
    return s


def run(s):
    kind = s["case"]["kind"]
    if kind == "era":
        sim = s["sim"]
        sim.restore(s["start"])
        sim.era_step()
        return dict(r=sim.ctx.r, v=sim.ctx.v, a=sim.ctx.a, t=sim.t, dt=sim.dt, dtc=sim.dtc)
    ctx = s["ctx"]
    if kind == "step":
        # (a second pass finds the active particles at the block time already: their
        # prediction and correction then leave the state as the first pass left it)
        ctx.predict(s["tb"])
        acc, _ = ctx.force(s["idx"], s["tb"], with_pot=False)
        ctx.correct(s["idx"], s["tb"], acc)
        dtc = ctx.timestep(s["idx"], ETA)
        return dict(acc=acc, dtc=dtc, r=ctx.r, v=ctx.v, a=ctx.a, t_last=ctx.t_last)
    if kind == "force":
        ctx.predict(s["tb"])
        acc, pot = ctx.force(s["idx"], s["tb"])
        return dict(acc=acc, pot=pot)
    if kind == "energy":
        return ctx.energy()
    if kind == "adjoint":
        gr, gm = ctx.force_backward(s["idx"], s["tb"], s["ga"], s["gp"])
        return dict(gr=gr, gm=gm)
    c = s["case"]
    if kind == "leapfrog":
        r, v = tsbts_leapfrog(s["r"], s["v"], s["m"], ctx, s["h"], c["steps"], c["era"])
    else:
        r, v = tsbts_block_leapfrog(s["r"], s["v"], s["m"], ctx, s["dt"], s["t_end"])
    grads = torch.autograd.grad([r, v], [s["r"], s["v"], s["m"]], [s["wr"], s["wv"]])
    return dict(r=r.detach(), v=v.detach(), gr=grads[0], gv=grads[1], gm=grads[2])


# ------------------------------------------------------------------ work
def _pairs(n, k):
    """Target-source pairs with those among the targets counted once: (both, one-sided)."""
    return k * (k - 1) / 2, k * (n - k)


def work(case):
    """Each input read and each output written once; the flops of the method's pair sums,
    a pair of two targets evaluated once for both (force 20 flops, 26 for both sides;
    criterion 15 and 20; adjoint 26 per part, 64 for both parts and sides; energy 12)."""
    n, kind = case["n"], case["kind"]
    state = 88 * n  # r, v, a, mass, last time of every particle
    if kind == "energy":
        return dict(bytes=56 * n + 16, flops=6 * n * (n - 1))
    if kind == "era":
        # every particle steps about once per smallest level in use in each pass; what
        # cannot be left out is one step of every particle per pass
        return dict(bytes=3 * 2 * state, flops=3 * 46 * n * (n - 1) / 2)
    if kind == "leapfrog":
        st = case["steps"]
        return dict(bytes=56 * n + 104 * n, flops=(26 * st + 64 * st) * n * (n - 1) / 2)
    if kind == "blocks":
        steps = 2 ** (case["levels"] - 1)
        flops = 0
        for s in range(1, steps + 1):
            due = min((s & -s).bit_length(), case["levels"])
            both, one = _pairs(n, n * due // case["levels"])
            flops += (26 + 64) * both + (20 + 52) * one
        return dict(bytes=56 * n + 104 * n, flops=flops)
    k = case["k"]
    both, one = _pairs(n, k)
    if kind == "step":
        return dict(bytes=state + 100 * k, flops=46 * both + 35 * one + 20 * n)
    if kind == "force":
        return dict(bytes=state + 36 * k, flops=26 * both + 20 * one + 20 * n)
    return dict(bytes=64 * n + 36 * k, flops=64 * both + 52 * one)


# ------------------------------------------------------------------ the same in float64
_CHUNK = 1 << 27  # pairs evaluated at a time


def _blocks(k, n):
    step = max(1, _CHUNK // n)
    return [slice(i, min(i + step, k)) for i in range(0, k, step)]


def _sep(rt, r, idx):
    """Separations [3][c, n] (source minus target) and the mask of the self pairs."""
    d = [r[c][None, :] - rt[c][:, None] for c in range(3)]
    return d, idx[:, None] == torch.arange(r.shape[1], device=r.device)[None, :]


def _force64(r, m, eps, idx):
    k, n = idx.numel(), r.shape[1]
    acc, pot = r.new_empty((3, k)), r.new_empty(k)
    for b in _blocks(k, n):
        d, own = _sep(r[:, idx[b]], r, idx[b])
        s = d[0] * d[0] + d[1] * d[1] + d[2] * d[2] + eps * eps
        y = s.masked_fill_(own, 1.0).rsqrt_().masked_fill_(own, 0.0)
        w = m[None, :] * y
        pot[b] = -w.sum(dim=1)
        w *= y * y
        for c in range(3):
            acc[c, b] = (w * d[c]).sum(dim=1)
    return acc, pot


def _criterion64(r, v, m, eps, idx):
    k, n = idx.numel(), r.shape[1]
    out = r.new_empty(k)
    wgt = m ** (-2.0 / 3.0)
    for b in _blocks(k, n):
        d, own = _sep(r[:, idx[b]], r, idx[b])
        r2 = d[0] * d[0] + d[1] * d[1] + d[2] * d[2]
        u, _ = _sep(v[:, idx[b]], v, idx[b])
        q = (u[0] * u[0] + u[1] * u[1] + u[2] * u[2]) / r2
        q.masked_fill_(own, 0.0)
        sw = ((r2 + eps * eps) * wgt[None, :]).masked_fill_(own, math.inf)
        tcol = q.max(dim=1).values.reciprocal().sqrt()
        tff = sw.min(dim=1).values ** 0.75
        out[b] = ETA * torch.minimum(tcol, tff)
    return out


def _adjoint64(r, m, eps, idx, ga, gp):
    """dL/dr, dL/dm of the acceleration and potential of the targets idx."""
    k, n = idx.numel(), r.shape[1]
    gr, gm = torch.zeros_like(r), torch.zeros_like(m)
    for b in _blocks(k, n):
        d, own = _sep(r[:, idx[b]], r, idx[b])
        s = d[0] * d[0] + d[1] * d[1] + d[2] * d[2] + eps * eps
        y = s.masked_fill_(own, 1.0).rsqrt_().masked_fill_(own, 0.0)
        y3 = y * y * y
        u = ga[0][b][:, None] * d[0] + ga[1][b][:, None] * d[1] + ga[2][b][:, None] * d[2]
        coef = 3.0 * y3 * y * y * u
        gmass = (y3 * u).sum(dim=0)
        if gp is not None:  # the potential -m y: its gradient in the separation is m y^3 d
            coef -= gp[b][:, None] * y3
            gmass -= (gp[b][:, None] * y).sum(dim=0)
        gm += gmass
        for c in range(3):
            t = m[None, :] * (y3 * ga[c][b][:, None] - coef * d[c])
            gr[c] += t.sum(dim=0)
            gr[c].index_add_(0, idx[b], -t.sum(dim=1))
    return gr, gm


def _leapfrog64(r, v, m, eps, times, sets):
    """Forward of a (block) leapfrog with every intermediate kept for the reverse sweep."""
    n = r.shape[1]
    every = torch.arange(n, device=r.device)
    a = _force64(r, m, eps, every)[0]
    t = torch.zeros(n, dtype=torch.float64, device=r.device)
    tape = []
    start = r
    for tb, idx in zip(times, sets):
        h = tb - t
        p = r + v * h + 0.5 * a * h * h
        an = _force64(p, m, eps, idx)[0]
        tape.append((p, h, idx))
        r, v, a, t = r.clone(), v.clone(), a.clone(), t.clone()
        r[:, idx] = p[:, idx]
        v[:, idx] += 0.5 * (a[:, idx] + an) * h[idx]
        a[:, idx] = an
        t[idx] = tb
    return start, r, v, tape


def _leapfrog_grad64(start, m, eps, tape, gr, gv):
    rb, vb = gr.clone(), gv.clone()
    ab, mb = torch.zeros_like(gr), torch.zeros_like(m)
    for p, h, idx in reversed(tape):
        pb = torch.zeros_like(rb)
        pb[:, idx] = rb[:, idx]
        rb[:, idx] = 0.0
        half = 0.5 * h[idx] * vb[:, idx]
        seed = ab[:, idx] + half
        ab[:, idx] = half
        dr, dm = _adjoint64(p, m, eps, idx, seed, None)
        pb += dr
        mb += dm
        rb += pb
        vb += pb * h
        ab += 0.5 * pb * h * h
    every = torch.arange(m.numel(), device=m.device)
    dr, dm = _adjoint64(start, m, eps, every, ab, None)
    return rb + dr, vb, mb + dm


def exact(case, seed):
    kind, n, eps = case["kind"], case["n"], case["eps"]
    if kind == "era":
        return None  # the steps are chosen along the way: a schedule, not a formula
    d = _inputs(case, seed)
    r, v, m = _gpu(d["r"]), _gpu(d["v"]), _gpu(d["m"])
    idx = torch.as_tensor(d["idx"], device="cuda").long() if "idx" in d else None
    if kind == "force":
        acc, pot = _force64(r, m, eps, idx)
        return dict(acc=acc, pot=pot)
    if kind == "step":
        a, t, tb = _gpu(d["a"]), _gpu(d["t_last"]), d["tb"]
        h = tb - t
        p, pv = r + v * h + 0.5 * a * h * h, v + a * h
        acc, _ = _force64(p, m, eps, idx)
        hk = h[idx]
        r2, v2, a2, t2 = r.clone(), v.clone(), a.clone(), t.clone()
        r2[:, idx] = p[:, idx]
        v2[:, idx] = v[:, idx] + 0.5 * (a[:, idx] + acc) * hk
        a2[:, idx] = acc
        t2[idx] = tb
        pv[:, idx] = v2[:, idx]
        return dict(acc=acc, dtc=_criterion64(p, pv, m, eps, idx), r=r2, v=v2, a=a2, t_last=t2)
    if kind == "energy":
        every = torch.arange(n, device="cuda")
        pot = _force64(r, m, eps, every)[1]
        return torch.stack([0.5 * (m * (v * v).sum(dim=0)).sum(), 0.5 * (m * pot).sum()])
    if kind == "adjoint":
        gr, gm = _adjoint64(r, m, eps, idx, _gpu(d["ga"]), _gpu(d["gp"]))
        return dict(gr=gr, gm=gm)
    every = torch.arange(n, device="cuda")
    if kind == "leapfrog":
        times = [(s + 1) * d["h"] for s in range(case["steps"])]
        sets = [every] * case["steps"]
    else:
        dt = _gpu(d["dt"])
        times = [(s + 1) * d["h"] for s in range(int(d["t_end"] / d["h"]))]
        sets = [torch.nonzero(torch.remainder(dt.new_tensor(t), dt) == 0).reshape(-1)
                for t in times]
    start, re, ve, tape = _leapfrog64(r, v, m, eps, times, sets)
    gr, gv, gm = _leapfrog_grad64(start, m, eps, tape, _gpu(d["wr"]), _gpu(d["wv"]))
    return dict(r=re, v=ve, gr=gr, gv=gv, gm=gm)
