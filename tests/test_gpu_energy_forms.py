"""Forms of the energies' near field (64 or 32 lanes per particle, or one) at
the sizes where one gives way to the next. All compute in FP64, and FP32C
contexts, without packed positions, keep to 32 lanes where FP64 ones take one:
the two agree within the bound of the energy terms against the oracle (1e-11),
and the small sizes with the oracle."""
import numpy as np
import pytest

import oracle
from gpu_common import system, to_device

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2609_02694_amd as rbe  # noqa: E402

TOL_E = 1e-11


def near_terms(p, s, prec, ncell=(0, 0, 0)):
    ctx = rbe.Context(rbe.params_from_preset(p, prec=prec, ncell=ncell,
                                             terms=rbe.TERM_LJ | rbe.TERM_COUL_REAL), len(s["x"]))
    u = ctx.energy(to_device(s), with_kinetic=False).cpu().numpy()
    ctx.sync_check()
    ctx.close()
    return u[[0, 1, 5, 6]]


@pytest.mark.parametrize("n", [4096, 4098])
def test_energy_groups_match_oracle(n):
    p, s = system("replica", n=n)
    u = near_terms(p, s, rbe.FP64)
    ref = oracle.real_energy(s["x"], s["y"], s["z"], s["q"], oracle.sys_from_preset(p))
    assert np.allclose(u[:2], ref, rtol=TOL_E, atol=0.0)


@pytest.mark.parametrize("name,n,over", [
    ("ljelectrolyte", 40_960, {}), ("ljelectrolyte", 40_962, {}),  # a nearly empty sphere
    ("replica", 196_608, {}), ("replica", 196_611, {}),            # a full one; a last tile of three particles
    ("replica", 200_000, {"frac_charged": 1.0}),
    ("replica", 200_000, {"frac_charged": 0.0}),
])
def test_energy_queue_matches_groups(name, n, over):
    p, s = system(name, n=n, **over)
    a, b = near_terms(p, s, rbe.FP64), near_terms(p, s, rbe.FP32C)
    print(f"energy forms {name} n={n} {over} rel {np.abs(a - b) / np.maximum(np.abs(b), 1e-300)}")
    assert np.allclose(a, b, rtol=TOL_E, atol=0.0)
