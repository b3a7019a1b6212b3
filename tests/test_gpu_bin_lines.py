"""Binning at the edges of its one-block forms: from positions (keys + 3 n up to
21,000, n^2 up to 180,000 keys) bit-exact against the oracle, and in a step from
keys (keys + n up to 13,000, n up to 8,192), which returns the particles in cell
order; and the buckets that are placed by counting (more than 8 entries, on
grids of fewer keys than half the particles)."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2609_02694_amd as rbe  # noqa: E402

L = 64.0


def particles(n, seed):
    rng = np.random.default_rng(seed)
    q = np.zeros(n)
    half = n // 3
    q[:half], q[half:2 * half] = 1.0, -1.0
    x, y, z = rng.uniform(0, L, (3, n))
    vx, vy, vz = rng.normal(size=(3, n))
    return dict(x=x, y=y, z=z, vx=vx, vy=vy, vz=vz, q=rng.permutation(q), id=np.arange(n, dtype=np.int32))


@pytest.mark.parametrize("n,ncell", [(6_600, (10, 10, 6)), (6_601, (10, 10, 6)), (500, (20, 20, 24)),
                                     (600, (20, 20, 24)), (601, (20, 20, 24)), (848, (2, 1, 1)), (849, (2, 1, 1)), (1, (1, 1, 1))])
def test_from_positions(n, ncell):
    s = particles(n, n)
    ctx = rbe.Context(rbe.make_params(L, 0.3, 1.0, 0.5, 4, ncell=ncell), n)
    for _ in range(2):
        cs, perm = ctx.build_cells(*(torch.as_tensor(s[k]).cuda() for k in ("x", "y", "z", "q")))
        cs_o, perm_o = oracle.bin_cells(s["x"], s["y"], s["z"], s["q"], L, ncell)
        assert np.array_equal(cs.cpu().numpy(), cs_o) and np.array_equal(perm.cpu().numpy(), perm_o)
    ctx.close()


@pytest.mark.parametrize("n,ncell", [(8_192, (8, 25, 12)), (8_193, (8, 25, 12)), (4_000, (20, 15, 15)),
                                     (4_001, (20, 15, 15)), (3, (50, 13, 10))])
def test_in_steps(n, ncell):
    ctx = rbe.Context(rbe.make_params(L, 0.3, 1.0, 0.5, 4, ncell=ncell, terms=rbe.TERM_FOURIER, dt=0.01), n)
    st = rbe.Particles.from_numpy(particles(n, n))
    ctx.forces(st)
    ctx.step(st, 3, 1)
    ctx.sync_check()
    ctx.close()
    got = {k: getattr(st, k).cpu().numpy() for k in ("x", "y", "z", "q", "id")}
    _, perm = oracle.bin_cells(got["x"], got["y"], got["z"], got["q"], L, ncell)
    assert np.array_equal(perm, np.arange(n)) and np.array_equal(np.sort(got["id"]), np.arange(n))


@pytest.mark.parametrize("n,ncell", [(20_000, (16, 16, 19)), (20_000, (16, 16, 20)),  # 2.06 and 1.95 particles a key
                                     (9_000, (16, 8, 8)),                           # buckets of about 8
                                     (70_000, (1, 1, 1)), (9_001, (2, 1, 1))])
@pytest.mark.parametrize("ordered", [False, True])
def test_long_buckets(n, ncell, ordered):
    s = particles(n, n)
    if ordered:
        _, o = oracle.bin_cells(s["x"], s["y"], s["z"], s["q"], L, ncell)
        s = {k: np.ascontiguousarray(v[o]) for k, v in s.items()}
    ctx = rbe.Context(rbe.make_params(L, 0.3, 1.0, 0.5, 4, ncell=ncell), n)
    cs, perm = ctx.build_cells(*(torch.as_tensor(s[k]).cuda() for k in ("x", "y", "z", "q")))
    cs_o, perm_o = oracle.bin_cells(s["x"], s["y"], s["z"], s["q"], L, ncell)
    ctx.close()
    assert np.array_equal(cs.cpu().numpy(), cs_o) and np.array_equal(perm.cpu().numpy(), perm_o)
