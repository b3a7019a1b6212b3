"""Random batch list, FP64: the group form (64 lanes per particle for a wide
shell, 32 or 16 for a narrow one) and the cluster form, at the sizes where one
gives way to the other. Against the oracle with the bounds of the other FP64
forms: 1e-12 over all particles, 1e-10 of the RMS force per row."""
import numpy as np
import pytest

import oracle
from gpu_common import ROW64, gpu_forces, max_row_err, rel_err, system

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2609_02694_amd as rbe  # noqa: E402


@pytest.mark.parametrize("name,n,over", [
    ("ljelectrolyte", 1_024, {}),                   # narrow shell, small grid
    ("ljelectrolyte", 2_000, {"r_core": 0.0001}),   # no core: all pairs in the shell
    ("ljelectrolyte", 8_192, {}),                   # narrow shell, the last size of 32 lanes
    ("ljelectrolyte", 8_194, {}),                   # and 16
    ("ljelectrolyte", 32_770, {}),
    ("ljelectrolyte", 65_536, {}),                  # the last size of the group form
    ("ljelectrolyte", 65_538, {}),                  # and the cluster form after it
    ("electrolyte1m", 9_001, {"ghost": 6.0}),       # wide shell, ghosts, a last group alone
    ("electrolyte1m", 9_001, {"p_shell": 32}),      # the longest batch
    ("electrolyte1m", (1 << 20) + 1, {}),           # wide shell, the cluster form
])
def test_rbl_forces_match_oracle(name, n, over):
    p, s = system(name, n=n, **over)
    rows = np.arange(0, n, 1 if n < 100_000 else 397)  # of the largest system a part
    for ev in (0, 5):
        F = gpu_forces(p, s, terms=rbe.TERM_LJ | rbe.TERM_COUL_REAL, ev=ev)[rows]
        ref = oracle.real_force(s["x"], s["y"], s["z"], s["q"], s["id"], oracle.sys_from_preset(p),
                                oracle.LJ | oracle.COUL_REAL, p["seed"], ev, idx=rows, cells=n > 5000)
        ref += (F - ref).mean(axis=0)  # the mean force, which the step takes off all rows
        e, r = rel_err(F, ref), max_row_err(F, ref)
        print(f"rbl {name} n={n} {over} ev={ev} rel err {e:.3e} max row {r:.3e}")
        assert e < 1e-12 and r < ROW64
