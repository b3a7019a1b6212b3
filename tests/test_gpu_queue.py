"""Queue walks of the FP64 near field (candidates filtered on packed 16-bit
positions) at the sizes that take them: parts above 65,536 neutral or 262,144
charged particles, batches above 262,144, and systems whose indices leave no
room for the image code of a queue entry. FP64 against the oracle to 1e-12."""
import numpy as np
import pytest

import gen
import oracle
from gpu_common import gpu_forces, oracle_forces, rel_err, system

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2609_02694_amd as rbe  # noqa: E402


@pytest.mark.parametrize("name,n,over,ncell", [
    ("subdomain64m", 75_001, {}, (0, 0, 0)),             # neutral part, ghost shell, a last wave that is not full
    ("subdomain64m", 75_001, {"ghost": 0.0}, (50, 9, 7)),  # periodic, uneven grid
    ("replica", 262_146, {"frac_charged": 1.0}, (0, 0, 0)),  # charged part
])
def test_queue_forces_match_oracle(name, n, over, ncell):
    p, s = system(name, n=n, **over)
    m, w = oracle.sample_k(p["seed"], 0, p["L"], p["alpha"], p["P"])
    ref = oracle_forces(p, s, m, w, terms=oracle.LJ | oracle.COUL_REAL, cells=True)
    F = gpu_forces(p, s, terms=rbe.TERM_LJ | rbe.TERM_COUL_REAL, m=m, w=w, ncell=ncell)
    e = rel_err(F, ref["lj"] + ref["coul"])
    print(f"queue {name} n={n} rel err {e:.3e}")
    assert e < 1e-12


def test_queue_batch_matches_single_contexts():
    """Replicas of a large FP64 batch (queue walk over several boxes per wave)
    against the same replicas alone (group walk): 1e-12 as above."""
    sizes = [1200] * 218 + [1013]
    reps, cat, off = gen.replica_batch(sizes)
    assert off[-1] > 262_144
    ctx = rbe.Context.batch([rbe.params_from_preset(p, seed=p["stream_seed"]) for p, _ in reps], off)
    st = rbe.Particles.from_numpy(cat)
    ctx.forces(st)
    ctx.sync_check()
    F = torch.stack([st.fx, st.fy, st.fz], 1).cpu().numpy()
    ctx.close()
    for r in (0, 100, 217, 218):
        p, s = reps[r]
        one = rbe.Context(rbe.params_from_preset(p, seed=p["stream_seed"]), sizes[r])
        st = rbe.Particles.from_numpy(s)
        one.forces(st)
        ref = torch.stack([st.fx, st.fy, st.fz], 1).cpu().numpy()
        one.close()
        assert rel_err(F[off[r]:off[r + 1]], ref) < 1e-12


def test_queue_without_room_for_the_image_code():
    """2^26 + 2 ions: the entries hold the index alone and the shift is the one
    of the row piece being scanned. Against the FP32C form (1e-5)."""
    n = (1 << 26) + 2
    p = gen.preset("plain3k", n=n)
    L, side = (n / (3000 / 30.0 ** 3)) ** (1 / 3), 407
    g = torch.Generator(device="cuda").manual_seed(3)
    site = torch.arange(n, device="cuda") * (side ** 3 // n)
    def axis(c):
        u = torch.rand(n, generator=g, device="cuda", dtype=torch.float64) - 0.5
        return (c + 0.5 + u) * (L / side)
    xyz = [axis(c) for c in (site % side, (site // side) % side, site // side ** 2)]
    del site
    q = 1.0 - 2.0 * (torch.arange(n, device="cuda", dtype=torch.float64) % 2)
    ids = torch.arange(n, device="cuda", dtype=torch.int32)
    f = []
    for prec in (rbe.FP64, rbe.FP32C):
        z = [torch.zeros(n, dtype=torch.float64, device="cuda") for _ in range(6)]
        st = rbe.Particles(*xyz, *z, q, ids)
        ctx = rbe.Context(rbe.make_params(L, p["alpha"], p["r_coul"], p["r_lj"], 1, prec=prec,
                                          terms=rbe.TERM_COUL_REAL), n)
        ctx.forces(st)
        ctx.sync_check()
        ctx.close()
        f.append(z[3:])
        del st, z
        torch.cuda.empty_cache()
    num = sum(float(((a - b) ** 2).sum()) for a, b in zip(*f))
    den = sum(float((a ** 2).sum()) for a in f[0])
    e = (num / den) ** 0.5
    print(f"queue n={n} rel diff to FP32C {e:.3e}")
    assert e < 1e-5
