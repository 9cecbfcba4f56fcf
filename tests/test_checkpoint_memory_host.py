"""What the checkpoints of a differentiated run hold (CPU stand-in context): positions,
velocities, accelerations and times of a run whose steps stay the same, the steps too of a
run on a recorded schedule."""
import numpy as np
import pytest
import torch

from workloads import plummer
from fake_context import FakeContext
from paper_1205_2288_amd.autograd import (fixed_schedule, tsbts_block_leapfrog,
                                          tsbts_leapfrog, tsbts_schedule_leapfrog)

N, H = 12, 1.0 / 64


def _run(kind):
    r, v, m = plummer(N, 31, masses="loguniform")
    x = [torch.tensor(a, requires_grad=True) for a in (r, v, m)]
    ctx = FakeContext(N, 1.0 / 16)
    dt = H * 2.0 ** (np.arange(N) % 2)
    if kind == "shared":
        return tsbts_leapfrog(*x, ctx, H, 6, 2)[0].grad_fn.checkpoints
    if kind == "block":
        return tsbts_block_leapfrog(*x, ctx, dt, 6 * H, 2)[0].grad_fn.checkpoints
    sched = fixed_schedule(dt, 6 * H, 2 * H, 2)
    return [(0, s) for s in tsbts_schedule_leapfrog(*x, ctx, sched)[0].grad_fn.starts]


@pytest.mark.parametrize("kind,values", [("shared", 10), ("block", 10), ("schedule", 11)])
def test_values_per_particle_of_a_checkpoint(kind, values):
    held = _run(kind)
    assert len(held) == 3
    assert all(flat.numel() == values * N for _, flat in held)
