"""Group walks of the near field (several lanes per particle) against the
oracle, at the sizes where their dispatch and their lists change: 64 lanes up
to 8,192 particles of a part and 32 above, chunks of 8 candidates per lane,
rows that cross the box edge, the ghost shell, species blocks of one particle.
Tolerances as in the parity tests: 1e-12 (FP64) and 1e-5 (FP32C) RMS."""
import numpy as np
import pytest

import gen
import oracle
from gpu_common import gpu_forces, oracle_forces, rel_err, system

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2609_02694_amd as rbe  # noqa: E402

PREC = [(rbe.FP64, 1e-12), (rbe.FP32C, 1e-5)]


@pytest.mark.parametrize("prec,tol", PREC)
@pytest.mark.parametrize("name,n,over", [
    ("replica", 868, {}),                   # smallest box: every row crosses its edge
    ("replica", 8192, {}),                  # the largest part of 64 lanes
    ("replica", 8194, {}),                  # 32 lanes
    ("replica", 8191, {"frac_charged": 2 / 8191}),  # two charged particles
    ("plain3k", 3000, {}),                  # an empty neutral part
    ("subdomain64m", 9000, {}),             # ghost shell, parts on both sides of 8,192
])
def test_group_forces_match_oracle(name, n, over, prec, tol):
    p, s = system(name, n=n, **over)
    m, w = oracle.sample_k(p["seed"], 0, p["L"], p["alpha"], p["P"])
    terms = rbe.TERM_LJ | rbe.TERM_COUL_REAL
    ref = oracle_forces(p, s, m, w, cells=False)
    F = gpu_forces(p, s, prec=prec, terms=terms, m=m, w=w)
    e = rel_err(F, ref["lj"] + ref["coul"])
    print(f"group {name} n={n} prec={prec} rel err {e:.3e}")
    assert e < tol


@pytest.mark.parametrize("prec,tol", PREC)
def test_group_lists_longer_than_a_chunk(prec, tol):
    """A cluster so dense that the rows of one round hold several chunks of
    candidates (512 at 64 lanes), beside empty space."""
    g = np.random.default_rng(5)
    n, L = 4000, 40.0
    side = np.arange(16)
    site = np.stack(np.meshgrid(side, side, side, indexing="ij"), -1).reshape(-1, 3)[:n]
    r = (18.0 + 0.55 * site + g.uniform(-0.02, 0.02, (n, 3))) % L  # about 6 per unit volume
    p = dict(gen.preset("plain3k", n=n), L=L, density=None)
    q = np.where(np.arange(n) % 2 == 0, 1.0, -1.0)
    s = dict(x=r[:, 0].copy(), y=r[:, 1].copy(), z=r[:, 2].copy(), q=q, id=np.arange(n, dtype=np.int32),
             vx=np.zeros(n), vy=np.zeros(n), vz=np.zeros(n))
    m, w = oracle.sample_k(p["seed"], 0, L, p["alpha"], p["P"])
    ref = oracle_forces(p, s, m, w, cells=False)
    F = gpu_forces(p, s, prec=prec, terms=rbe.TERM_COUL_REAL, m=m, w=w)
    e = rel_err(F, ref["coul"])
    print(f"group dense prec={prec} rel err {e:.3e}")
    assert e < tol


def test_group_fp32c_bits_do_not_depend_on_the_lanes():
    """FP32C: a row's terms are summed in order whatever the number of lanes,
    so a system computes the same bits alone (64 lanes per particle) and as a
    member of a batch whose size takes 32 lanes or one thread per particle."""
    p = gen.preset("replica", n=2000)
    s = gen.make_system(p)
    ncell = (18, 6, 6)
    base = dict(ncell=ncell, prec=rbe.FP32C, terms=rbe.TERM_COUL_REAL)
    alone = rbe.Context(rbe.params_from_preset(p, seed=1, **base), 2000)
    st = rbe.Particles.from_numpy(s)
    alone.forces(st)
    ref = torch.stack([st.fx, st.fy, st.fz]).cpu().numpy()
    alone.close()
    for copies in (8, 70):
        cat = {k: np.concatenate([v] * copies) for k, v in s.items() if k != "L"}
        off = [2000 * k for k in range(copies + 1)]
        ctx = rbe.Context.batch([rbe.params_from_preset(p, seed=k, **base) for k in range(copies)], off)
        st = rbe.Particles.from_numpy(cat)
        ctx.forces(st)
        ctx.sync_check()
        F = torch.stack([st.fx, st.fy, st.fz]).cpu().numpy()
        for k in range(copies):
            assert np.array_equal(F[:, off[k]:off[k + 1]], ref), (copies, k)
        ctx.close()
