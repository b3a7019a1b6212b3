"""Plain sums of sparse systems (21 particles within the reach, and 5) at the
sizes where the group walk gives way to one thread per particle: 65,536 and
32,768 charged particles in FP64, 32,768 in FP32C. 1e-12 (FP64) and 1e-5 (FP32C) RMS."""
import pytest

import oracle
from gpu_common import gpu_forces, rel_err, system

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2609_02694_amd as rbe  # noqa: E402


@pytest.mark.parametrize("n,prec,tol", [(32_768, rbe.FP64, 1e-12), (32_770, rbe.FP64, 1e-12),
                                        (65_536, rbe.FP64, 1e-12), (65_538, rbe.FP64, 1e-12),
                                        (32_768, rbe.FP32C, 1e-5), (32_770, rbe.FP32C, 1e-5)])
@pytest.mark.parametrize("terms,r", [(oracle.COUL_REAL, 8.0), (oracle.LJ | oracle.COUL_REAL, 8.0),
                                     (oracle.LJ | oracle.COUL_REAL, 5.0)])
def test_sparse_forces_match_oracle(n, prec, tol, terms, r):
    p, s = system("ljelectrolyte", n=n, r_core=0.0, r_coul=r, r_lj=r)
    F = gpu_forces(p, s, prec=prec, terms=terms)
    ref = oracle.real_force(s["x"], s["y"], s["z"], s["q"], s["id"], oracle.sys_from_preset(p), terms, cells=True)
    e = rel_err(F, ref)
    print(f"sparse n={n} prec={prec} terms={terms} rel err {e:.3e}")
    assert e < tol
