"""Multi-vector float64 products at the edges of their tiles (64, 128 and 256 spheres by system
size) and for every count of vectors left over from the launches of four, each vector against
the ordered single-vector kernel: the same float64 terms in another order, so within 1e-13
(sqrt(n) 2^-53 ~ 2e-14 at the largest n here)."""
import numpy as np
import pytest

from paper_1612_00474_amd import workloads as wl
from tests.gpu_util import close, dev, host, require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,nvec", [(1, 3), (65, 2), (127, 5), (6999, 1), (7001, 3), (28001, 2)])
@pytest.mark.parametrize("wall", [True, False])
def test_multi_tile_edges(n, nvec, wall):
    require_gpu()
    from paper_1612_00474_amd import Context
    c = Context(0, wall=wall)
    pos = wl.sheet(n, 0.8, 2.6, seed=n)
    F = dev(np.random.default_rng(n).standard_normal((nvec, n, 3)))
    u = host(c.matvec_multi(dev(pos), F, "fp64"))
    c.set_tuning("fp64", symmetric=0)
    for v in range(nvec):
        assert close(u[v], host(c.matvec(dev(pos), F[v], None, "fp64")), 1e-13), (n, v, wall)
    c.close()
