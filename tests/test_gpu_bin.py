"""Binning at the sizes where its forms give way to one another: one block up
to 8,192 particles and 32,768 keys; the scan without a pass of its own over the
tiles' sums up to 1,024 tiles of 2,048 keys. Bit-exact against the oracle, twice
on one context (the second call finds what the first left)."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2609_02694_amd as rbe  # noqa: E402


@pytest.mark.parametrize("n,ncell,one_cell", [
    (1, (3, 3, 3), False), (1023, (4, 4, 4), False), (1025, (4, 4, 4), True),
    (8192, (8, 8, 8), False), (8193, (8, 8, 8), False),
    (8192, (32, 32, 16), False), (5000, (32, 32, 17), False),              # the most keys of the block, and more
    (3000, (128, 64, 128), False), (3000, (128, 65, 128), False),          # 1,024 tiles, and more
])
def test_bin_forms_bit_exact(n, ncell, one_cell):
    L, rng = 64.0, np.random.default_rng(n)
    params = rbe.make_params(L, 0.3, 1.0, 0.5, 4, ncell=ncell)
    ctx = rbe.Context(params, n)
    for _ in range(2):
        x, y, z = rng.uniform(0, 0.1 if one_cell else L, (3, n))
        q = rng.integers(-1, 2, n).astype(np.float64)
        cs, perm = ctx.build_cells(*(torch.as_tensor(a).cuda() for a in (x, y, z, q)))
        cs_o, perm_o = oracle.bin_cells(x, y, z, q, L, ncell)
        assert np.array_equal(cs.cpu().numpy(), cs_o) and np.array_equal(perm.cpu().numpy(), perm_o)
    ctx.close()


@pytest.mark.parametrize("n", [1200, 9000])
def test_steps_in_one_call_equal_single_steps(n):
    """The histogram of a call's later steps is the one its scatter cleared."""
    import gen
    p = gen.preset("replica", n=n)
    s = gen.make_system(p)
    out = []
    for calls in ((4,), (1, 1, 2)):
        ctx = rbe.Context(rbe.params_from_preset(p), n)
        st, ev = rbe.Particles.from_numpy(s), 1
        ctx.forces(st, None, None, 0)
        for k in calls:
            ctx.step(st, k, ev)
            ev += k
        ctx.sync_check()
        ctx.close()
        o = np.argsort(st.id.cpu().numpy())
        out.append(np.stack([getattr(st, a).cpu().numpy()[o] for a in ("x", "y", "z", "vx", "vy", "vz")]))
    assert np.allclose(out[0], out[1], rtol=0, atol=1e-9)
