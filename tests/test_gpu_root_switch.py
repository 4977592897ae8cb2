"""The switch of the tridiagonal root between its quadrature and the eigendecomposition: leading
blocks that are safely positive definite up to some order and singular, nearly singular or
indefinite from there on, so that one sequence uses both and the eigendecomposition is brought up
from order 1 at the first block that needs it.  Against LAPACK's eigendecomposition.

Tolerance: T^{1/2} moves by eps |T| / (2 lambda_min^{1/2}) under a rounding of T where it is definite,
so rows are compared within 64 eps (|T| / lambda_min)^{1/2} (at most 1e-12 where lambda_min is at
least 1e-6 |T|), and within (64 eps)^{1/2} of |T|^{1/2}, the root's modulus of continuity, where it is
smaller."""
import numpy as np
import pytest

from tests.gpu_util import require_gpu

pytestmark = pytest.mark.gpu


def _ref(alpha, beta):
    T = np.diag(alpha) + np.diag(beta, 1) + np.diag(beta, -1)
    lam, Q = np.linalg.eigh(T)
    return (Q * np.sqrt(np.maximum(lam, 0.0))) @ Q[0], lam


@pytest.mark.parametrize("m", [1, 2, 7, 8, 9, 16, 17, 32, 33, 64])
@pytest.mark.parametrize("kind", ["definite", "singular_end", "near_singular", "indefinite_mid",
                                  "scaled_up", "scaled_down"])
def test_root_switch(m, kind):
    require_gpu()
    from paper_1612_00474_amd import Context
    rng = np.random.default_rng(m)
    alpha, beta = rng.uniform(1.5, 3.0, m), rng.uniform(0.1, 0.7, m - 1)
    if kind == "singular_end":        # last pivot zero
        d = alpha[0]
        for i in range(1, m):
            d = alpha[i] - beta[i - 1] ** 2 / d
        alpha[-1] -= d
    elif kind == "near_singular":
        alpha[m // 2] = 1e-9
        if m > 1:
            beta[max(0, m // 2 - 1):m // 2 + 1] = 1e-7
    elif kind == "indefinite_mid":
        alpha[m // 2] = -0.5
    elif kind == "scaled_up":
        alpha, beta = alpha * 1e120, beta * 1e120
    elif kind == "scaled_down":
        alpha, beta = alpha * 1e-60, beta * 1e-60
    c = Context(0)
    got = c.tridiag_sqrt(alpha, beta, 1.7)
    c.close()
    eps = np.finfo(float).eps
    for k in range(1, m + 1):
        ref, lam = _ref(alpha[:k], beta[:k - 1])
        top = np.abs(lam).max()
        ratio = lam[0] / top
        tol = min(64 * eps / np.sqrt(ratio), 1e-12) if ratio >= 1e-6 else np.sqrt(64 * eps)
        assert np.linalg.norm(got[k - 1, :k] - 1.7 * ref) <= 1.7 * tol * np.sqrt(top), (m, kind, k)
        assert not got[k - 1, k:].any()
