"""Fourier kernels at the sizes where their forms give way to one another: mode
counts around the blocks of eight modes and the waves of 64 that share a
chunk's particles, particle counts around a wave and at the last size whose
gather is shared by the waves of a block. Against the oracle: FP64 to 1e-12,
FP32C to 1e-5, as for the whole force."""
import numpy as np
import pytest

import oracle
from gpu_common import ROW32, ROW64, max_row_err, rel_err, to_device

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2609_02694_amd as rbe  # noqa: E402


@pytest.mark.parametrize("prec,tol,row", [(rbe.FP64, 1e-12, ROW64), (rbe.FP32C, 1e-5, ROW32)])
@pytest.mark.parametrize("n,P", [
    (2, 1), (63, 7), (64, 8), (65, 9), (66, 63), (130, 64), (130, 65), (514, 127), (514, 128), (514, 129), (514, 136),
    (1000, 1023), (1000, 1024), (1000, 2050),                       # and the modes split over groups
    (196_608, 20), (196_610, 20), (262_144, 20), (262_146, 20),
])
def test_fourier_forms_match_oracle(prec, tol, row, n, P):
    L, alpha, rng = 20.0, 0.3, np.random.default_rng(n + P)
    s = {k: rng.uniform(0, L, n) for k in "xyz"} | {k: np.zeros(n) for k in ("vx", "vy", "vz")}
    s |= {"q": np.where(np.arange(n) % 2, -1.0, 1.0) * (np.arange(n) < n - n % 2), "id": np.arange(n, dtype=np.int32)}
    m, w = oracle.sample_k(7, 0, L, alpha, P)
    ctx = rbe.Context(rbe.make_params(L, alpha, 1.0, 1.0, P, prec=prec, terms=rbe.TERM_FOURIER), n)
    st, rho = to_device(s), torch.zeros(2 * P, dtype=torch.float64, device="cuda")
    ctx.forces(st, torch.as_tensor(np.ascontiguousarray(m, np.int32).ravel()).cuda(), torch.as_tensor(w).cuda(), 0, rho)
    ctx.sync_check()
    ctx.close()
    F = torch.stack([st.fx, st.fy, st.fz], 1).cpu().numpy()
    rho = rho.cpu().numpy()
    re, im = oracle.rho(s["x"], s["y"], s["z"], s["q"], L, m)
    ref, _, _ = oracle.fourier_force(s["x"], s["y"], s["z"], s["q"], L, m, w, re, im)
    e, r = rel_err(F, ref), max_row_err(F, ref)
    print(f"fourier forms n={n} P={P} prec={prec} rel err {e:.3e} max row {r:.3e}")
    assert e < tol and r < row
    tol_rho = 1e-12 if prec == rbe.FP64 else 1e-6
    assert max(np.abs(rho[:P] - re).max(), np.abs(rho[P:] - im).max()) < tol_rho * np.sqrt(n)
