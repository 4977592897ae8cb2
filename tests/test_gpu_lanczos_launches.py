"""The launch forms of the Lanczos vector work: one or four elements per thread, the root taken by
the update or by a launch of its own, the one-workgroup form of small systems, and the host
reading the flags late, each by a batch that takes it (empty and one-sphere systems among them)
against the single-system solve of the same rows.

Tolerance: the same Krylov process in float64 with sums in another order, 1e-11 on the increment
at tol 1e-6 (each of ~30 iterations adds rounding of a few 1e-16, amplified by the condition of
T^{1/2}, at most ~1e2 here); the iteration counts are equal."""
import numpy as np
import pytest

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


@pytest.mark.parametrize("sizes", [
    [300, 0, 1, 512],                    # one workgroup per system
    [513, 0, 1, 85, 86],                 # one element per thread, root in the update
    [700] + [40] * 100,                  # four elements per thread, root in the update
    [700] + [20] * 300 + [0, 1],         # root in a launch of its own
])
def test_batched_forms(ctx, sizes):
    offs = np.concatenate([[0], np.cumsum(sizes)])
    pos = np.vstack([wl.sheet(n, 0.9, 2.5, seed=i) for i, n in enumerate(sizes) if n])
    w = np.random.default_rng(len(sizes)).standard_normal(pos.shape)
    g, it, eps, st = ctx.lanczos_batched(dev(pos), offs, dev(w), 1e-6, 64)
    g = host(g)
    again = host(ctx.lanczos_batched(dev(pos), offs, dev(w), 1e-6, 64)[0])
    assert st == 0 and np.array_equal(g, again)
    for s in sorted({0, 1, 2, 3, len(sizes) - 1}):
        a, b = offs[s], offs[s + 1]
        if a == b:
            continue
        one, m, e, _ = ctx.lanczos(dev(pos[a:b]), dev(w[a:b]), 1e-6)
        assert it[s] == m and close(g[a:b], host(one), 1e-11), (s, it[s], m)


@pytest.mark.parametrize("n", [200, 1100, 4097])   # one workgroup; flags read late; flags read at once
def test_multi_forms(ctx, n):
    pos = wl.sheet(n, 0.9, 2.5, seed=n)
    w = np.random.default_rng(n).standard_normal((5, n, 3))
    w[3] *= 1e-3
    g, it, eps, st = ctx.lanczos_multi(dev(pos), dev(w), 1e-3)
    for v in range(5):
        one, m, e, _ = ctx.lanczos(dev(pos), dev(w[v]), 1e-3)
        assert it[v] == m and close(host(g)[v], host(one), 1e-11), (v, it[v], m)


@pytest.mark.parametrize("n", [21845, 21846, 43700, 174763])   # edges of 256 and 512 workgroups
def test_single_forms(ctx, n):
    if n > 100000:   # the vector work alone: two mixed iterations
        pos, tol, it_max, precision = wl.sheet(n, 1.1, 2.5, seed=1), 1e-300, 2, "mixed"
    else:
        pos, tol, it_max, precision = wl.sheet(n, 1.1, 2.5, seed=1), 1e-300, 4, "fp64"
    w = dev(np.random.default_rng(n).standard_normal((n, 3)))
    p = dev(pos)
    g, m, _, _ = ctx.lanczos(p, w, tol, it_max, precision=precision, allow_noconv=True)
    # the Krylov iterate from the library's products and plain vector algebra
    import torch
    norm = float(w.norm())
    basis, alpha, beta = [w / norm], [], []
    for _ in range(it_max):
        u = ctx.matvec(p, basis[-1], None, precision)
        alpha.append(float((u * basis[-1]).sum()))
        for _ in range(2):
            for v in basis:
                u = u - (u * v).sum() * v
        beta.append(float(u.norm()))
        basis.append(u / beta[-1])
    T = np.diag(alpha) + np.diag(beta[:-1], 1) + np.diag(beta[:-1], -1)
    lam, Q = np.linalg.eigh(T)
    y = norm * (Q * np.sqrt(lam)) @ Q[0]
    ref = sum(float(c) * v for c, v in zip(y, basis))
    assert m == it_max and close(host(g), host(ref), 1e-12 if precision == "fp64" else 1e-7)


def test_flags_of_earlier_contexts():
    """A new context's pinned flag words hold nothing of an earlier context's solves."""
    require_gpu()
    from paper_1612_00474_amd import Context
    pos = dev(wl.sheet(60, 1.1, 2.5, seed=2))
    w = dev(np.random.default_rng(2).standard_normal((6, 60, 3)))
    first = None
    for _ in range(4):
        c = Context(0)
        for _ in range(6):
            g, it, _, _ = c.lanczos_multi(pos, w, 1e-300, 5, allow_noconv=True)
            first = host(g) if first is None else first
            assert list(it) == [5] * 6 and np.array_equal(host(g), first)
        c.close()
