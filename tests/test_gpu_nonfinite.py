"""Forces beside particles whose position is not finite: such a particle is
within no cutoff of any other and no member of their shells, so the others'
forces are those of the system without it (the oracle's), and its own pair
terms are zero."""
import numpy as np
import pytest

import oracle
from gpu_common import ROW64, gpu_forces, max_row_err, rel_err, system

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2609_02694_amd as rbe  # noqa: E402


@pytest.mark.parametrize("name,n,over", [
    ("electrolyte1m", 4_000, {}),               # wide shell: 64 lanes per particle
    ("electrolyte1m", 4_000, {"ghost": 6.0}),
    ("ljelectrolyte", 3_000, {}),               # narrow shell, charged particles out of it
    ("replica", 3_000, {}),                     # plain sums
])
def test_other_particles_do_not_see_it(name, n, over):
    p, s = system(name, n=n, **over)
    bad = np.flatnonzero(s["q"] == 0)[:3] if (s["q"] == 0).any() else np.arange(3)
    s["x"][bad[0]] = np.nan
    s["y"][bad[1]] = np.inf
    for k in "xyz":
        s[k][bad[2]] = np.nan
    F = gpu_forces(p, s, terms=rbe.TERM_LJ | rbe.TERM_COUL_REAL)
    keep = np.setdiff1d(np.arange(n), bad)
    ref = np.zeros((n, 3))
    ref[keep] = oracle.real_force(*(s[k][keep] for k in ("x", "y", "z", "q", "id")), oracle.sys_from_preset(p),
                                  oracle.LJ | oracle.COUL_REAL, p["seed"], 0)
    if p["r_core"] > 0:
        ref -= ref.mean(axis=0)
    e, r = rel_err(F, ref), max_row_err(F, ref)
    print(f"non-finite {name} n={n} {over} rel err {e:.3e} max row {r:.3e}")
    assert e < 1e-12 and r < ROW64
