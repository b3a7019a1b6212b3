"""Random batch list, FP64: the forms by the size of a part (32 lanes per
particle or clusters, both launched) and the mean force (Eq. 12), which the
library takes off all rows: the reference is corrected by its own mean, and of
the systems too large for a reference of every row the sum of the forces is
checked as well. 1e-12 over all rows, 1e-10 of the RMS force per row."""
import numpy as np
import pytest

import oracle
from gpu_common import ROW64, gpu_forces, max_row_err, rel_err, system

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2609_02694_amd as rbe  # noqa: E402


def reference(p, s, rows, ev):
    return oracle.real_force(s["x"], s["y"], s["z"], s["q"], s["id"], oracle.sys_from_preset(p),
                             oracle.LJ | oracle.COUL_REAL, p["seed"], ev, idx=rows, cells=len(s["x"]) > 5000)


@pytest.mark.parametrize("name,n,over", [
    ("ljelectrolyte", 2_000, {}), ("ljelectrolyte", 9_000, {}), ("ljelectrolyte", 66_000, {}),
    ("electrolyte1m", 9_001, {}), ("electrolyte1m", 9_001, {"ghost": 6.0}),
    ("electrolyte1m", 65_538, {"r_coul": 5.0}),                # wide shell, the first size of 32 lanes
])
def test_forces_and_mean(name, n, over):
    p, s = system(name, n=n, **over)
    for ev in (0, 5):
        F, ref = gpu_forces(p, s, terms=rbe.TERM_LJ | rbe.TERM_COUL_REAL, ev=ev), reference(p, s, np.arange(n), ev)
        ref -= ref.mean(axis=0)
        e, r = rel_err(F, ref), max_row_err(F, ref)
        print(f"rbl {name} n={n} {over} ev={ev} rel err {e:.3e} max row {r:.3e}")
        assert e < 1e-12 and r < ROW64


@pytest.mark.parametrize("n,over", [
    (270_002, {}),                                       # a full shell: 64 lanes
    (270_002, {"r_coul": 5.0}),                          # 32 lanes, launched beside the clusters
    (270_002, {"r_coul": 5.0, "frac_charged": 1.0}),     # clusters
    (270_002, {"r_coul": 5.0, "frac_charged": 0.02, "r_lj": 4.0}),  # the neutral part takes the list too
    (270_002, {"r_coul": 5.0, "ghost": 5.0}),
    (393_218, {}),                                       # a full shell, 32 lanes
    # cells as wide as the reach: clusters from parts of 65,537 on
    (83_002, {"r_coul": 4.0, "r_lj": 4.0, "frac_charged": 0.5}),
    (83_002, {"r_coul": 4.0, "r_lj": 4.0, "frac_charged": 1.0}),
    (90_002, {"r_coul": 4.0, "r_lj": 4.0, "frac_charged": 0.05}),
    (100_002, {"r_coul": 4.0, "r_lj": 4.0, "frac_charged": 1.0, "ghost": 4.0}),
])
def test_parts_of_a_large_system(n, over):
    p, s = system("electrolyte1m", n=n, **over)
    rows = np.arange(0, p["n"], 61)
    F = gpu_forces(p, s, terms=rbe.TERM_LJ | rbe.TERM_COUL_REAL, ev=3)
    frms = np.sqrt((F ** 2).sum() / len(F))
    assert np.abs(F.mean(axis=0)).max() < 1e-12 * frms
    ref = reference(p, s, rows, 3)
    ref += (F[rows] - ref).mean(axis=0)  # the mean over all rows
    e, r = rel_err(F[rows], ref), max_row_err(F[rows], ref)
    print(f"rbl parts {over} rel err {e:.3e} max row {r:.3e}")
    assert e < 1e-12 and r < ROW64
