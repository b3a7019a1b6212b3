"""FP32C near field: the rows a walk closes are part of the result, so the
thread form (batches above 131,072 particles) and the group form (a small system
alone) close the same ones and give the same bits."""
import numpy as np
import pytest

import gen

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2609_02694_amd as rbe  # noqa: E402


def test_thread_and_group_forms_same_bits():
    sizes = [1200] * 110
    reps, cat, off = gen.replica_batch(sizes)
    kw = dict(prec=rbe.FP32C, terms=rbe.TERM_COUL_REAL)
    ctx = rbe.Context.batch([rbe.params_from_preset(p, seed=p["stream_seed"], **kw) for p, _ in reps], off)
    st = rbe.Particles.from_numpy(cat)
    ctx.forces(st)
    ctx.sync_check()
    F = torch.stack([st.fx, st.fy, st.fz], 1).cpu().numpy()
    ctx.close()
    for r in range(0, len(sizes), 9):
        p, s = reps[r]
        one = rbe.Context(rbe.params_from_preset(p, seed=p["stream_seed"], **kw), sizes[r])
        st = rbe.Particles.from_numpy(s)
        one.forces(st)
        ref = torch.stack([st.fx, st.fy, st.fz], 1).cpu().numpy()
        one.close()
        assert np.array_equal(F[off[r]:off[r + 1]], ref)
