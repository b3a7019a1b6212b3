"""FP32C near field: the rows a walk closes are those its FP64 reach touches.
The walks choose rows in single precision, with the reach enlarged by some
2^-18; an empty row closed for the enlargement's sake would add a zero to the
Kahan sums, which moves their rounding where a row's sum exceeds the sum so far.

Clusters far apart, each a target particle with neighbours in the rows below,
beside and above it along z; the target sits 2e-5 farther than the cutoff from
the next row along y, which is empty and is visited before the rows above. On a
grid of wider cells along y that row is far out of reach and everything else is
the same, so the forces agree to the last bit."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2609_02694_amd as rbe  # noqa: E402

R, HY = 3.0, 8.0  # cutoff, narrow cells along y (the wide ones: 12)


@pytest.mark.parametrize("clusters", [400, 2_600])  # group walk; one thread per particle
def test_row_just_out_of_reach(clusters):
    g = np.random.default_rng(7)
    shape = (clusters, 13)
    x = 12.0 * np.arange(clusters)[:, None] + 6.0 + g.uniform(-1.5, 1.5, shape)
    y = g.uniform(3.3, 4.6, shape)
    row = np.repeat([5, 4, 5, 6], [1, 4, 4, 4])  # z-rows of edge 1.9; a target is within reach of both neighbours' rows
    z = 1.9 * row + g.uniform(0.1, 1.8, shape)
    y[:, 0], z[:, 0] = HY - R - 2e-5, 1.9 * 5 + 0.95
    q = g.uniform(0.3, 1.5, (clusters // 2, 13)) * g.choice([-1.0, 1.0], (clusters // 2, 13))
    q = np.stack([q, -q], axis=1).reshape(shape)
    s = {k: v.ravel() for k, v in dict(x=x, y=y, z=z, q=q).items()}
    n = x.size
    F = []
    for ny in (6, 4):
        params = rbe.make_params((12.0 * clusters, 48.0, 19.0), 0.3, R, 1.0, 1, prec=rbe.FP32C,
                                 ncell=(8 * clusters, ny, 10), terms=rbe.TERM_COUL_REAL)
        ctx = rbe.Context(params, n)
        st = rbe.Particles.from_numpy(dict(s, id=np.arange(n, dtype=np.int32)))
        ctx.forces(st)
        F.append(torch.stack([st.fx, st.fy, st.fz]).cpu().numpy())
        ctx.close()
    assert np.array_equal(F[0], F[1])
