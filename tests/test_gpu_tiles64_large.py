"""Float64 tiles of 512 spheres (from 96,000 on), the only ones larger than the sources staged at a
time: ragged last tiles that end in the first and in the second stage, one sphere into it, and
full, against the ordered kernel on rows around the tile edges and at both ends.

Tolerance: the same float64 terms in another order, sqrt(n) 2^-53 ~ 4e-14."""
import numpy as np
import pytest

from paper_1612_00474_amd import workloads as wl
from tests.gpu_util import close, dev, host, require_gpu

pytestmark = pytest.mark.gpu

TILE, STAGE = 512, 256


@pytest.mark.parametrize("n", [188 * TILE - 1, 187 * TILE + STAGE + 1, 188 * TILE + 100, 188 * TILE])
@pytest.mark.parametrize("torque", [False, True])
def test_ragged_large_tiles(n, torque):
    require_gpu()
    from paper_1612_00474_amd import Context
    c = Context(0)
    assert n >= 96_000
    rng = np.random.default_rng(n)
    pos, F, T = dev(wl.sheet(n, 0.8, 2.6, seed=n)), *map(dev, rng.standard_normal((2, n, 3)))
    t = T if torque else None
    u = host(c.matvec(pos, F, t, "fp64"))
    last = (n - 1) // TILE * TILE
    for a, b in ((0, 130), (TILE - 3, TILE + 3), (40 * TILE + STAGE - 3, 40 * TILE + STAGE + 3),
                 (last - 70, n)):
        assert close(u[a:b], host(c.matvec(pos, F, t, "fp64", rows=(a, b))), 1e-13), (a, b)
    c.close()
