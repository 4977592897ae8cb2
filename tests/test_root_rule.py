"""CPU: the rule that hands a tridiagonal to the eigendecomposition (a pivot of the elimination from the
last row below 1e-8 of the Gershgorin bound) holds for every larger leading block once it holds for
one, so a solve need not try the quadrature again."""
import numpy as np


def _left(a, b):
    """Whether the rule leaves diag a, off-diagonal b to the eigendecomposition."""
    m = len(a)
    e = np.zeros(m)
    e[:-1] += np.abs(b)
    e[1:] += np.abs(b)
    bound = np.max(np.abs(a) + e)
    d = a[-1]
    smallest = d
    for i in range(m - 2, -1, -1):
        if not smallest >= 1e-8 * bound:
            return True
        d = a[i] - b[i] * b[i] / d
        smallest = min(smallest, d)
    return not smallest >= 1e-8 * bound


def test_left_once_left_ever():
    rng = np.random.default_rng(0)
    switches = 0
    for trial in range(3000):
        m = int(rng.integers(2, 41))
        kind = trial % 4
        if kind == 0:      # indefinite somewhere
            a, b = rng.standard_normal(m) + rng.uniform(0, 3), rng.uniform(0, 1, m - 1)
        elif kind == 1:    # a Gram matrix of graded vectors: nearly singular
            lo, d = rng.uniform(0, 2, m - 1), 10.0 ** rng.uniform(-9, 1, m)
            a = d.copy()
            a[:-1] += lo * lo * d[1:]
            b = lo * d[1:]
        elif kind == 2:    # positive definite, growing
            a, b = 2.1 + rng.uniform(0, 3, m) * np.arange(m), rng.uniform(0, 1, m - 1)
        else:              # the second difference, shifted towards zero
            a, b = np.full(m, 2.0 - rng.uniform(0, 0.1)), np.ones(m - 1)
        left = [_left(a[:k], b[:k - 1]) for k in range(1, m + 1)]
        first = left.index(True) if True in left else m
        assert all(left[first:]), (trial, left)
        switches += 0 < first < m
    assert switches > 500   # the rule switched inside the sequence often enough to mean something
