"""Steps on a grid of many more cells than particles: the histogram of a call's
later steps is the one that its scatter cleared, by more threads than particles."""
import numpy as np
import pytest

import gen

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2609_02694_amd as rbe  # noqa: E402


@pytest.mark.parametrize("n,ncell", [(900, (64, 64, 64)), (900, (128, 128, 100)), (9_000, (40, 40, 40))])
def test_steps_in_one_call_equal_single_steps(n, ncell):
    p = gen.preset("replica", n=n)
    s = gen.make_system(p)
    out = []
    for calls in ((4,), (1, 1, 2)):
        ctx = rbe.Context(rbe.params_from_preset(p, terms=rbe.TERM_FOURIER, ncell=ncell), n)
        st, ev = rbe.Particles.from_numpy(s), 1
        ctx.forces(st, None, None, 0)
        for k in calls:
            ctx.step(st, k, ev)
            ev += k
        ctx.sync_check()
        ctx.close()
        out.append([getattr(st, a).cpu().numpy() for a in ("id", "x", "y", "z", "vx", "vy", "vz")])
    assert all(np.array_equal(a, b) for a, b in zip(*out))
