"""Mode tables with columns (FP64): the kernels that take a segment of up to
nine modes of one (m_x, m_y) at a time against those that take any mode, which
serve the same table in an order that leaves no columns. Both evaluate every
phase in FP64 (at most 80 turns a component here), so rows agree to 1e-12 and
structure factors to 1e-12 of sqrt(sum q^2), as with the oracle."""
import numpy as np
import pytest

from gpu_common import ROW64, max_row_err, rel_err, to_device

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2609_02694_amd as rbe  # noqa: E402


def columns(lengths, rng, aligned=False):
    """Columns of the given lengths at random (m_x, m_y, first m_z)."""
    out = []
    for k in lengths:
        mx, my, mz = rng.integers(-20, 21, 3)
        out += [(mx, my, (9 * (mz // 9) if aligned else mz) + j) for j in range(k)]
    return np.array(out, np.int32).T


def table(kind, L):
    rng = np.random.default_rng(5)
    if kind == "lattice":
        return rbe.lattice_modes(rbe.make_params(L, 0.9, 3.0, 1.0, 1), 6.0)
    m = {"lengths": lambda: columns(list(range(1, 92)), rng),          # every remainder of nine, singles among them
         "short": lambda: columns([3] * 1400, rng),                    # fewer than 4 modes a segment: none are cut
         "four": lambda: columns([4] * 1100, rng, True),               # exactly 4: the most segments there is room for
         "least": lambda: columns([64] * 64, rng),                     # the shortest table
         "below": lambda: columns([64] * 63 + [63], rng),              # too short a table
         "repeats": lambda: np.concatenate([columns([70] * 30, rng)] * 2, axis=1),
         "descending": lambda: columns(list(range(1, 92)), rng)[:, ::-1]}[kind]()
    return m, rng.uniform(0.1, 1.0, m.shape[1]) / m.shape[1]


@pytest.mark.parametrize("kind", ["lattice", "lengths", "short", "four", "least", "below", "repeats", "descending"])
@pytest.mark.parametrize("n", [1, 16, 17, 700, 4001])
def test_segments_match_the_general_kernels(kind, n):
    L = (11.0, 12.5, 17.0)
    m, w = table(kind, L)
    rng = np.random.default_rng(n)
    q = np.where(np.arange(n) % 2, -1.0, 1.0) * (np.arange(n) < n - n % 2)  # neutral, an odd one uncharged
    s = {k: rng.uniform(0, L[d], n) for d, k in enumerate("xyz")}
    s |= {k: np.zeros(n) for k in ("vx", "vy", "vz")} | {"q": q, "id": np.arange(n, dtype=np.int32)}
    P = m.shape[1]
    ctx = rbe.Context(rbe.make_params(L, 0.9, 3.0, 1.0, P, kc=1.7, terms=rbe.TERM_FOURIER), n)
    got = []
    for how in ("mixed", "call", "fixed"):
        order = rng.permutation(P) if how == "mixed" else np.arange(P)
        md = torch.as_tensor(np.ascontiguousarray(m[:, order]).ravel()).cuda()
        wd = torch.as_tensor(np.ascontiguousarray(w[order])).cuda()
        if how == "fixed":
            ctx.set_modes(md, wd)
            md = wd = None
        st, rho = to_device(s), torch.zeros(2 * P, dtype=torch.float64, device="cuda")
        ctx.forces(st, md, wd, 0, rho)
        u = ctx.energy(st, md, wd)
        ctx.sync_check()
        r = np.empty((2, P))
        r[:, order] = rho.cpu().numpy().reshape(2, P)
        got.append((torch.stack([st.fx, st.fy, st.fz], 1).cpu().numpy(), r, u.cpu().numpy()))
    ctx.close()
    (f0, r0, u0), (f1, r1, u1), (f2, r2, u2) = got
    assert rel_err(f1, f0) < 1e-12 and max_row_err(f1, f0) < ROW64
    assert np.abs(r1 - r0).max() <= 1e-12 * max(1.0, np.sqrt((q ** 2).sum()))
    assert np.allclose(u1, u0, rtol=1e-12, atol=1e-14)
    assert np.array_equal(f2, f1) and np.array_equal(r2, r1) and np.array_equal(u2, u1)


def test_segments_follow_the_table():
    """A later table, a call's own one and the way back to drawing each take
    the place of the segments before."""
    L, n, P = 12.0, 500, 4200
    rng = np.random.default_rng(2)
    s = {k: rng.uniform(0, L, n) for k in "xyz"} | {k: np.zeros(n) for k in ("vx", "vy", "vz")}
    s |= {"q": np.where(np.arange(n) % 2, -1.0, 1.0), "id": np.arange(n, dtype=np.int32)}
    ctx = rbe.Context(rbe.make_params(L, 0.9, 3.0, 1.0, P, terms=rbe.TERM_FOURIER, seed=4), n)

    def forces(*args):
        st = to_device(s)
        ctx.forces(st, *args)
        return torch.stack([st.fx, st.fy, st.fz], 1).cpu().numpy()

    def device(m):
        return torch.as_tensor(np.ascontiguousarray(m).ravel()).cuda()

    drawn = forces()
    own = device(columns([60] * 70, rng)), torch.as_tensor(rng.uniform(0.1, 1.0, P)).cuda()
    first = forces(*own)
    for lengths in ([40] * 105, [3] * 1400, [100] * 42):
        m, w = columns(lengths, rng), rng.uniform(0.1, 1.0, P)
        order = rng.permutation(P)
        ref = forces(device(m[:, order]), torch.as_tensor(w[order]).cuda())
        ctx.set_modes(device(m), torch.as_tensor(w).cuda())
        assert rel_err(forces(), ref) < 1e-12
        assert np.array_equal(forces(*own), first)
        assert rel_err(forces(), ref) < 1e-12
    ctx.set_modes(None, None)
    assert np.array_equal(forces(), drawn)
    ctx.close()
