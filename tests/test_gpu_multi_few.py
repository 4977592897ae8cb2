"""Multi-vector float64 products of a few spheres: the rotation steps of the tile kernel at which no two
of them meet are left out."""
import numpy as np
import pytest

from oracle import mobility
from paper_1612_00474_amd import workloads as wl
from tests.gpu_util import close, dev, host, require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    require_gpu()
    from paper_1612_00474_amd import Context
    c = Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("n", [1, 2, 3, 16, 31, 32, 33, 34, 48, 63, 64, 66, 97])
@pytest.mark.parametrize("nvec", [1, 4])
def test_every_pair_is_met_once(ctx, n, nvec):
    pos = wl.sheet(n, 0.8, 2.6, seed=n)
    F = np.random.default_rng(n).standard_normal((nvec, n, 3))
    u = host(ctx.matvec_multi(dev(pos), dev(F), "fp64"))
    for v in range(nvec):
        assert close(u[v], mobility.dense_matvec(pos, F[v], None), 1e-12), (n, v)
        single = host(ctx.matvec(dev(pos), dev(F[v]), None, "fp64"))
        assert close(u[v], single, 1e-13), (n, v)


def test_one_sphere_takes_less_than_a_tile(ctx):
    def launch_us(n):
        pos = dev(wl.sheet(n, 1.1, 2.5, seed=n))
        F = dev(np.random.default_rng(n).standard_normal((4, n, 3)))
        ctx.matvec_multi(pos, F, "fp64")
        ctx.timing(True)
        ctx.timing_read()
        for _ in range(50):
            ctx.matvec_multi(pos, F, "fp64")
        ms, launches, _ = ctx.timing_read(8)
        ctx.timing(False)
        return 1e3 * ms / launches

    # every step evaluated, both took 17 us between their events
    assert launch_us(1) < 0.8 * launch_us(64)
