"""Single Lanczos solves whose vector work takes one workgroup (preconditioned ones, and launch shapes
other than the small solve's own), at the sizes where the form changes."""
import numpy as np
import pytest

from oracle import lanczos, mobility
from paper_1612_00474_amd import workloads as wl
from tests.gpu_util import close, dev, host, require_gpu

pytestmark = pytest.mark.gpu

# fixed iterations: the same Krylov space, rounding of the products
TOL = {"fp64": 1e-12, "mixed": 1e-5}


def _case(n):
    pos = wl.sheet(n, 0.8, 2.6, seed=n)
    return pos, np.random.default_rng(n).standard_normal((n, 3)), mobility.dense(pos)[0]


@pytest.mark.parametrize("n,m", [(2, 4), (85, 12), (86, 5), (256, 24), (257, 6), (512, 12), (513, 6)])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_preconditioned(n, m, precision):
    require_gpu()
    from paper_1612_00474_amd import Context
    pos, w, M = _case(n)
    c = Context(0)
    ref, mref, _, _ = lanczos.lanczos_sqrt_precond(lambda v: M @ v, lanczos.block_diagonal_scale(pos),
                                                   w.ravel(), 1e-300, m)
    g, it, _, _ = c.lanczos(dev(pos), dev(w), 1e-300, m, precision, allow_noconv=True, precond=True)
    c.close()
    assert it == mref == m
    assert close(host(g).ravel(), ref, TOL[precision])


@pytest.mark.parametrize("n,precision,shape", [(200, "fp64", dict(symmetric=0)),
                                               (257, "fp64", dict(symmetric=0)),
                                               (300, "mixed", dict(tpt=1)),
                                               (512, "mixed", dict(tpt=1)),
                                               (300, "mixed", dict(symmetric=0))])
def test_other_launch_shapes(n, precision, shape):
    require_gpu()
    from paper_1612_00474_amd import Context
    pos, w, M = _case(n)
    c = Context(0)
    c.set_tuning(precision, **shape)
    for m in (1, 9, 33):
        ref, mref, _, _ = lanczos.lanczos_sqrt(lambda v: M @ v, w.ravel(), 1e-300, m)
        g, it, _, _ = c.lanczos(dev(pos), dev(w), 1e-300, m, precision, allow_noconv=True)
        assert it == mref == m
        assert close(host(g).ravel(), ref, TOL[precision]), m
    # stopped by its tolerance, the same solve capped there, and a step from it
    g, it, eps, _ = c.lanczos(dev(pos), dev(w), 1e-4, 64, precision)
    capped, it2, eps2, _ = c.lanczos(dev(pos), dev(w), 1e-4, it, precision)
    assert (it2, eps2) == (it, eps) and np.array_equal(host(g), host(capped))
    c.close()


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_exhausted_space(precision):
    require_gpu()
    from paper_1612_00474_amd import Context
    pos, w, M = _case(1)
    c = Context(0)
    g, it, _, _ = c.lanczos(dev(pos), dev(w), 1e-300, 64, precision, precond=True)
    c.close()
    assert it <= 3
    assert close(host(g).ravel(), lanczos.sqrtm_dense(M) @ w.ravel(), 10 * TOL[precision])
