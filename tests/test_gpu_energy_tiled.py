"""Energies of a periodic system and of the same system repeated twice along
every axis, whose near terms are eight times those of the one: the one small
enough for the group walk (checked against the oracle elsewhere), the other so
large that one lane takes a particle, in either precision of the context."""
import numpy as np
import pytest

from gpu_common import system

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2609_02694_amd as rbe  # noqa: E402


@pytest.mark.parametrize("prec", [rbe.FP64, rbe.FP32C])
@pytest.mark.parametrize("name,n,over", [
    ("ljelectrolyte", 6_000, {}),                   # a nearly empty sphere
    ("replica", 24_601, {}),                        # a full one, charged and neutral particles
    ("replica", 24_601, {"r_lj": 6.0}),             # the LJ terms reach as far as the Coulomb terms
    ("replica", 24_600, {"frac_charged": 0.0}),
    ("electrolyte1m", 24_601, {}),
])
def test_tiled_system(name, n, over, prec):
    p, s = system(name, n=n, **over)
    u = []
    for c in (1, 2):
        k = np.arange(c ** 3)
        shift = dict(x=k % c, y=k // c % c, z=k // c ** 2)
        t = {a: (s[a][None, :] + shift[a][:, None] * p["L"]).ravel() for a in "xyz"}
        t["q"], t["id"] = np.tile(s["q"], c ** 3), np.arange(n * c ** 3, dtype=np.int32)
        params = rbe.params_from_preset(dict(p, L=c * p["L"]), prec=prec, terms=rbe.TERM_LJ | rbe.TERM_COUL_REAL)
        ctx = rbe.Context(params, n * c ** 3)
        u.append(ctx.energy(rbe.Particles.from_numpy(t), with_kinetic=False).cpu().numpy()[[0, 1, 5, 6]])
        ctx.sync_check()
        ctx.close()
    print(f"tiled {name} prec={prec} rel {np.abs(u[1] / 8 - u[0]) / np.maximum(np.abs(u[0]), 1e-300)}")
    assert np.allclose(u[1], 8 * u[0], rtol=1e-11, atol=0.0)
