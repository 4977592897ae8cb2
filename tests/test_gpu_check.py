"""The finite check of the positions travels with their packing, and the product is enqueued before
its verdict is read: a NaN or Inf in any workgroup of any size must end in RPB_ENONFINITE with the
output untouched, and must leave nothing behind for the next call."""
import numpy as np
import pytest

from paper_1612_00474_amd import workloads as wl
from tests.gpu_util import dev, host, require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("n", [1, 255, 256, 257, 1500, 70000])
def test_non_finite_positions_leave_the_output_alone(n, precision):
    require_gpu()
    import torch
    from paper_1612_00474_amd import Context
    from paper_1612_00474_amd._lib import RPB_ENONFINITE, RpbError
    c = Context(0)
    pos = wl.sheet(n, 0.8, 2.6, seed=n)
    P = dev(pos)
    F = dev(np.random.default_rng(n).standard_normal((3, n, 3)))
    calls = {"matvec": lambda q, out: c.matvec(q, F[0], F[1], precision, out=out),
             "torque": lambda q, out: c.matvec(q, None, F[1], precision, out=out)}
    if n < 70000:
        calls["rows"] = lambda q, out: c.matvec(q, F[0], None, precision, out=out, rows=(0, n // 2 + 1))
        calls["multi"] = lambda q, out: c.matvec_multi(q, F, precision, out=out)
        calls["lanczos"] = lambda q, out: c.lanczos(q, F[0], 1e-3, 64, precision, out=out)
    for name, call in calls.items():
        shape = {"rows": (n // 2 + 1, 3), "multi": (3, n, 3)}.get(name, (n, 3))
        out = torch.empty(shape, dtype=torch.float64, device="cuda")
        call(P, out)
        good = host(out)
        for row, value in ((0, float("nan")), (n - 1, float("inf")), (n // 2, -float("inf"))):
            bad = P.clone()
            bad[row, row % 3] = value
            out.fill_(7.0)
            with pytest.raises(RpbError) as e:
                call(bad, out)
            assert e.value.status == RPB_ENONFINITE, name
            assert (host(out) == 7.0).all(), (name, row)
            call(P, out)
            assert np.array_equal(host(out), good), (name, row)
    c.close()
