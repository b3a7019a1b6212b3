"""LJ cell tiles of the FP32C form at odd particle counts, where the last lanes
and blocks of a tile are short: 8, 2 and 1 lanes per particle, with and without
the ghost shell. Against the oracle to 1e-5 as for the other FP32C forms."""
import pytest

import oracle
from gpu_common import ROW32, gpu_forces, max_row_err, oracle_forces, rel_err, system

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2609_02694_amd as rbe  # noqa: E402


@pytest.mark.parametrize("name,n,over", [
    ("replica", 869, {}), ("replica", 2_001, {}), ("replica", 24_001, {}), ("replica", 50_001, {}),
    ("replica", 90_001, {}),
    ("subdomain64m", 9_001, {}), ("subdomain64m", 30_001, {}), ("subdomain64m", 45_001, {}),
    ("subdomain64m", 9_001, {"ghost": 0.0}),
])
def test_odd_counts_match_oracle(name, n, over):
    p, s = system(name, n=n, **over)
    m, w = oracle.sample_k(p["seed"], 0, p["L"], p["alpha"], p["P"])
    ref = oracle_forces(p, s, m, w, terms=oracle.LJ, cells=True)["F"]
    F = gpu_forces(p, s, prec=rbe.FP32C, terms=rbe.TERM_LJ, m=m, w=w)
    e, r = rel_err(F, ref), max_row_err(F, ref)
    print(f"tile lanes {name} n={n} rel err {e:.3e} max row {r:.3e}")
    assert len(s["x"]) == n and e < 1e-5 and r < ROW32
