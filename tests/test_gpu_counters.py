"""The count of tested candidates means the same in every form of the near
field: a particle's own record is one of its candidates."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2609_02694_amd as rbe  # noqa: E402


@pytest.mark.parametrize("side,frac,prec", [
    (4, 0.5, rbe.FP64), (4, 0.5, rbe.FP32C),  # group walk
    (41, 0.0, rbe.FP64),                      # queue walk
    (41, 1.0, rbe.FP32C),                     # one thread per particle
])
def test_lone_particles_test_themselves_alone(side, frac, prec):
    n, a = side ** 3, 20.0
    site = np.arange(n)
    x, y, z = ((np.asarray(k) + 0.5) * a for k in (site % side, site // side % side, site // side ** 2))
    half = int(n * frac) // 2
    q = np.zeros(n)
    q[:half], q[half:2 * half] = 1.0, -1.0
    # cells of edge 4, the cutoff 3: every particle sits in the middle of a cell
    params = rbe.make_params(side * a, 1.0, 3.0, 3.0, 1, prec=prec, ncell=(5 * side,) * 3,
                             terms=rbe.TERM_COUL_REAL if frac == 1.0 else rbe.TERM_LJ | rbe.TERM_COUL_REAL)
    ctx = rbe.Context(params, n)
    ctx.set_counting(True)
    st = rbe.Particles.from_numpy(dict(x=x, y=y, z=z, q=q, id=np.arange(n, dtype=np.int32)))
    ctx.forces(st)
    cnt = ctx.counters()
    # without LJ terms the one neutral particle has no pair to test
    assert sum(c[2] for c in cnt.values()) == (2 * half if frac == 1.0 else n)
    assert all(c[0] == c[1] == 0 for c in cnt.values())
    ctx.close()
