"""The random finite difference evaluates its two products from one packing launch and, in float64,
in one pair launch: the same kernels as two separate products at pos +- (delta/2) w, so the drift
must equal their scaled difference to the bit, at the sizes where the tile changes and where the
partials of one product fit the workspace limit but not those of two."""
import numpy as np
import pytest

from paper_1612_00474_amd import workloads as wl
from tests.gpu_util import dev, host, require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rfd_precision", ["fp64", "mixed"])
@pytest.mark.parametrize("n,kib", [(1, 0), (65, 0), (300, 60), (1499, 0), (1500, 0), (6001, 0),
                                   (24001, 0)])
def test_drift_is_the_difference_of_two_products(n, kib, rfd_precision, monkeypatch):
    require_gpu()
    from paper_1612_00474_amd import Context
    if kib:
        monkeypatch.setenv("RPB_CHUNK_KIB", str(kib))
    c = Context(0)
    pos = wl.sheet(n, 0.8, 2.6, seed=n)
    w = np.random.default_rng(n).standard_normal((n, 3))
    delta = 1e-4
    for one_sided in (False, True):
        sp, sm = (delta, 0.0) if one_sided else (0.5 * delta, 0.5 * delta)
        up = host(c.matvec(dev(pos + sp * w), dev(w), None, rfd_precision))
        um = host(c.matvec(dev(pos - sm * w), dev(w), None, rfd_precision))
        got = host(c.rfd(dev(pos), dev(w), delta, precision=rfd_precision,
                         rfd_precision=rfd_precision,
                         rfd_scheme="one_sided" if one_sided else "centred"))
        assert np.array_equal(got, (c.kT / delta) * (up - um)), (n, one_sided)
    c.close()


def test_float64_tuning_keeps_to_shapes_that_serve_the_drift():
    # four targets per lane are the float64 products' own choice by size already, and the
    # slowest shape of the drift of mixed steps, so the tuner does not offer them
    require_gpu()
    from paper_1612_00474_amd import Context
    c = Context(0)
    pos = wl.sheet(4500, seed=1)
    c.autotune(dev(pos), precision="fp64")
    assert c.tuning()["fp64"]["tpt"] in (1, 2)
    c.close()
