"""GPU: the launch-shape tuner's float64 choice for single systems."""
import numpy as np
import pytest

from tests.gpu_util import dev, require_gpu

pytestmark = pytest.mark.gpu


def _sheet(n):
    from paper_1612_00474_amd import workloads as wl
    return dev(wl.sheet(n, 1.1, 2.5, seed=n))


@pytest.mark.parametrize("sizes", [(6001,), (8191,), (16384,), (4099, 8191), (8191, 4099, 6001)])
@pytest.mark.parametrize("wall", [True, False])
def test_float64_tile_is_not_cut_down(sizes, wall):
    """From 6,000 spheres on one target per lane makes the float64 tile smaller and the product slower,
    so the tuner keeps the launch of the default shape, whatever it was asked for before."""
    require_gpu()
    from paper_1612_00474_amd import Context
    c = Context(0, wall=wall)
    for n in sizes:
        shape, _ = c.autotune(_sheet(n), None, "fp64")
        if n >= 6000:
            assert (shape["symmetric"], shape["tpt"]) == (1, 2), (n, shape)
    c.close()
