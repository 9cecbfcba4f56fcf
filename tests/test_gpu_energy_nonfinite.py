"""Energy of a set whose last particle has an infinite velocity: the kinetic energy is
infinite (not undefined through the lanes past the last particle), the potential unchanged."""
import numpy as np
import pytest

from workloads import plummer
from gpu_util import make_ctx

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 255, 256, 300, 4097])
def test_infinite_velocity_of_the_last_particle(n):
    r, v, m = plummer(n, 8500 + n, masses="loguniform")
    ctx = make_ctx(n, 1 / 64, "fp64")
    ctx.bind(r, v, m)
    pot = ctx.energy().cpu().numpy()[1]
    v[1, n - 1] = np.inf
    ctx.bind(r, v, m)
    kin, again = ctx.energy().cpu().numpy()
    ctx.close()
    assert kin == np.inf and again == pot
