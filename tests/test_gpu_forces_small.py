"""Forces around the sizes where the wavefront-per-target kernel starts, ends a workgroup and hands
over to the cell list (6,000 spheres, 3,000 in a box), against the oracle.  Both sum the same
float64 terms; a pair's term is off by the rounding of r over b in the exponential (about
6 2^-52 / 0.1 < 2e-14) and a few of its neighbours' cancel, so 1e-13 of the norm."""
import numpy as np
import pytest

from oracle import forces
from paper_1612_00474_amd import workloads as wl
from tests.gpu_util import close, dev, host, require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("box", [False, True])
@pytest.mark.parametrize("n", [1, 2, 4, 5, 64, 65, 2999, 3000, 3001, 6000, 6001])
def test_forces_around_the_kernel_edges(n, box):
    require_gpu()
    from paper_1612_00474_amd import Context
    side = max(14.0, np.sqrt(n * np.pi / 0.4))   # more than two cutoffs of 6 a
    rng = np.random.default_rng(n)
    pos = np.column_stack([rng.uniform(0, side, n), rng.uniform(0, side, n),
                           rng.uniform(0.8, 2.6, n)])
    rows = np.unique(np.concatenate([np.arange(min(n, 200)), np.arange(max(0, n - 200), n)]))
    for wall in (True, False):
        c = Context(0, wall=wall, box=(side, side) if box else None)
        got = host(c.forces(dev(pos), -1.0, 1.0, 0.1))
        ref = forces.forces(pos, 1.0, 1.0, 0.1, -1.0, rows=rows, wall=wall,
                            box=(side, side) if box else None)
        assert close(got[rows], ref, 1e-13), (n, box, wall)
        c.close()
