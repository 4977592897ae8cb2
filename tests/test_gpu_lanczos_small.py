"""The one-launch-per-iteration Lanczos of small systems (up to 512 spheres) at the edges of its
workgroups (12 rows), thread counts (256 spheres fill one value per thread) and register blocks
(16 and 32 basis vectors), with a wall, in free space and in a box, against the Krylov iterate that
plain vector algebra makes of the library's own products.

Tolerance: float64 1e-11 (sums in another order, as in the batched comparison); mixed 1e-7: both
sides form the same float32 sums from v_k, whose elements agree to 1e-15, so only a source that
rounds the other way (6e-8 of one element) can differ."""
import numpy as np
import pytest
import torch

from paper_1612_00474_amd import workloads as wl
from tests.gpu_util import close, dev, host, require_gpu

pytestmark = pytest.mark.gpu


def _plain(ctx, pos, w, m, precision):
    norm = float(w.norm())
    basis, alpha, beta = [w / norm], [], []
    for _ in range(m):
        u = ctx.matvec(pos, basis[-1], None, precision)
        alpha.append(float((u * basis[-1]).sum()))
        for _ in range(2):
            for v in basis:
                u = u - (u * v).sum() * v
        beta.append(float(u.norm()))
        basis.append(u / beta[-1])
    T = np.diag(alpha) + np.diag(beta[:-1], 1) + np.diag(beta[:-1], -1)
    lam, Q = np.linalg.eigh(T)
    y = norm * (Q * np.sqrt(np.maximum(lam, 0.0))) @ Q[0]
    return sum(float(c) * v for c, v in zip(y, basis))


@pytest.mark.parametrize("n,m", [(4, 3), (11, 5), (12, 16), (13, 17), (255, 9), (256, 33),
                                 (257, 18), (341, 2), (512, 33), (513, 6)])
@pytest.mark.parametrize("kind", ["wall", "free", "box"])
@pytest.mark.parametrize("precision,tpt", [("fp64", 2), ("mixed", 1), ("mixed", 2), ("mixed", 4)])
def test_small_lanczos(n, m, kind, precision, tpt):
    require_gpu()
    from paper_1612_00474_amd import Context
    side = max(wl.side_for_area_fraction(n, 0.3), 8.0)
    c = Context(0, wall=kind != "free", box=(2 * side, 2 * side) if kind == "box" else None)
    c.set_tuning(precision, tpt=tpt)
    pos = dev(wl.sample_positions(n, side, 1.1, 3.0, seed=n))
    w = dev(np.random.default_rng(n).standard_normal((n, 3)))
    g, it, _, _ = c.lanczos(pos, w, 1e-300, m, precision=precision, allow_noconv=True)
    again = c.lanczos(pos, w, 1e-300, m, precision=precision, allow_noconv=True)[0]
    ref = _plain(c, pos, w, m, precision)
    c.close()
    assert it == m and torch.equal(g, again)
    assert close(host(g), host(ref), 1e-11 if precision == "fp64" else 1e-7), (n, m, kind)
