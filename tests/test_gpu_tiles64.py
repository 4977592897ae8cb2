"""The float64 symmetric tile kernels at the edges of their tiles: systems one sphere short of, equal
to and one past a multiple of the 64-sphere blocks and of every tile the size rule picks, with
and without torque, against the ordered kernel of the same call (an independent pair function and
summation order) and, where it is small enough, the oracle.

Tolerance: both are float64 sums of n terms whose sizes fall off with distance; against the
oracle the bound is the 1e-12 of every float64 product, against the ordered kernel 1e-13 (the
same terms, other rounding: sqrt(n) 2^-53 ~ 2e-14 at the largest n here)."""
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


@pytest.mark.parametrize("n", [1, 63, 65, 129, 1499, 1501, 5999, 6001, 11999, 12001, 24001])
@pytest.mark.parametrize("torque", [False, True])
def test_tile_edges(ctx, n, torque):
    pos = wl.sheet(n, 0.8, 2.6, seed=n)
    rng = np.random.default_rng(n)
    F, T = rng.standard_normal((2, n, 3))
    args = (dev(pos), dev(F), dev(T) if torque else None, "fp64")
    ref = mobility.dense_matvec(pos, F, T if torque else np.zeros_like(T)) if n < 200 else None
    for tpt in (1, 2):
        ctx.set_tuning("fp64", symmetric=1, tpt=tpt)
        u = host(ctx.matvec(*args))
        assert np.array_equal(u, host(ctx.matvec(*args)))   # reproducible
        if ref is not None:
            assert close(u, ref, 1e-12), (n, torque, tpt)
        ctx.set_tuning("fp64", symmetric=0)
        assert close(u, host(ctx.matvec(*args)), 1e-13), (n, torque, tpt)
    ctx.set_tuning("fp64", symmetric=1, tpt=2)
