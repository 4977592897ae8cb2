"""The float64 drift of mixed-precision steps: two products in one launch (the default) against the
same two in launches of their own (a workspace limit that holds one product's partials, 24 (parts +
1) bytes per tile pair and row of a tile, but not two), to the bit."""
import numpy as np
import pytest

from paper_1612_00474_amd import workloads as wl
from tests.gpu_util import dev, host, require_gpu

pytestmark = pytest.mark.gpu


def _one_product_kib(n, tpt):
    """Partials of one product: tiles of 256 tpt spheres, their sources split for small systems."""
    ts = 256 * tpt
    nt = -(-n // ts)
    pairs, parts = nt * (nt + 1) // 2, 1
    while pairs * parts < 4096 and ts // (2 * parts) >= 128:
        parts *= 2
    while pairs * parts < 64 and ts // (2 * parts) >= 8:
        parts *= 2
    return -(-pairs * (parts + 1) * 3 * ts * 8 // 1024)


@pytest.mark.parametrize("tpt", [1, 2])
@pytest.mark.parametrize("n", [1, 300, 513, 1501, 6001])
@pytest.mark.parametrize("box", [False, True])
def test_paired_drift_is_the_unpaired_one(n, tpt, box, monkeypatch):
    require_gpu()
    from paper_1612_00474_amd import Context
    pos = dev(wl.sheet(n, 0.8, 2.6, seed=n))
    w = dev(np.random.default_rng(n).standard_normal((n, 3)))
    side = max(8.0, wl.side_for_area_fraction(n, 0.4))

    def drift():
        c = Context(0, box=(side, side)) if box else Context(0)
        c.set_tuning("fp64", tpt=tpt)
        d = host(c.rfd(pos, w, 1e-4, precision="mixed", rfd_precision="fp64"))
        c.close()
        return d

    both = drift()
    one = _one_product_kib(n, tpt)
    monkeypatch.setenv("RPB_CHUNK_KIB", str(max(64, one + one // 2)))
    assert np.array_equal(drift(), both)
