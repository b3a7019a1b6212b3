"""Where one form of a kernel gives way to another, a call costs no more than
its neighbours on the other side of the line. Times are the best of several
runs and are compared with each other only, with room for their scatter."""
import time

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2609_02694_amd as rbe  # noqa: E402


def best_us(fn, reps=20, rounds=9):
    """Best time of fn in microseconds over rounds of reps calls."""
    best = float("inf")
    for _ in range(rounds + 1):  # the first one warms up
        torch.cuda.synchronize()
        t = time.perf_counter()
        for _ in range(reps):
            fn()
        torch.cuda.synchronize()
        best = min(best, (time.perf_counter() - t) / reps)
    return 1e6 * best


def random_state(n, L, charged=1.0, seed=5):
    """Particles on randomly occupied lattice sites, displaced by up to 0.15 of the lattice constant, in random order."""
    g = np.random.default_rng(seed)
    side = int(np.ceil(n ** (1 / 3) - 1e-9))
    site = g.permutation(side ** 3)[:n]
    r = [(np.asarray(k) + 0.5 + g.uniform(-0.15, 0.15, n)) * (L / side)
         for k in (site % side, site // side % side, site // side ** 2)]
    half = int(n * charged) // 2
    q = np.zeros(n)
    q[:half], q[half:2 * half] = 1.0, -1.0
    return rbe.Particles.from_numpy(dict(x=r[0], y=r[1], z=r[2], q=g.permutation(q), id=np.arange(n, dtype=np.int32)))


def test_binning_on_a_grid_of_many_more_cells_than_particles():
    """16 million keys: binning 300 particles takes no longer than 50,000."""
    t, params = {}, rbe.make_params(400.0, 0.3, 2.0, 1.0, 4, ncell=(200, 200, 200))
    for n in (300, 50_000):
        ctx, st = rbe.Context(params, n), random_state(n, 400.0)
        t[n] = best_us(lambda: ctx.build_cells(st.x, st.y, st.z, st.q))
        ctx.close()
    print(f"binning, 16M keys: {t}")
    assert t[300] < 1.3 * t[50_000]


@pytest.mark.parametrize("n,ncell", [(300, (32, 32, 15)), (4_000, (32, 32, 15)), (8_000, (16, 16, 16)),
                                     (8_000, (32, 32, 15))])
def test_binning_in_one_block(n, ncell):
    """A grid just small enough for the sort in one block so far, against one too large for it in any case."""
    t = {}
    for nc in (ncell, (32, 32, 40)):
        ctx, st = rbe.Context(rbe.make_params(96.0, 0.3, 2.0, 1.0, 4, ncell=nc), n), random_state(n, 96.0)
        t[nc] = best_us(lambda: ctx.build_cells(st.x, st.y, st.z, st.q))
        ctx.close()
    print(f"binning of {n}: {t}")
    assert t[ncell] < 1.15 * t[32, 32, 40]


@pytest.mark.parametrize("n,ncell", [(900, (32, 32, 15)), (8_000, (32, 32, 15))])
def test_steps_binned_in_one_block(n, ncell):
    """The same for the binning of a step, from keys (Fourier part alone: the grid matters to nothing else)."""
    t = {}
    for nc in (ncell, (32, 32, 40)):
        params = rbe.make_params(96.0, 0.3, 2.0, 1.0, 4, ncell=nc, terms=rbe.TERM_FOURIER, dt=1e-6)
        ctx, st = rbe.Context(params, n), random_state(n, 96.0)
        ctx.forces(st)
        t[nc] = best_us(lambda: ctx.step(st, 10, 1), reps=4)
        ctx.close()
    print(f"10 steps of {n}: {t}")
    assert t[ncell] < 1.1 * t[32, 32, 40]


@pytest.mark.parametrize("n,m", [(120_000, 3), (600_000, 3), (600_000, 60)])
def test_energy_of_a_single_precision_context(n, m):
    """Energies are summed in FP64 whatever the context's precision: the call costs the same."""
    t, r = {}, (m / (4.0 / 3.0 * np.pi * 0.1)) ** (1 / 3)
    L = (n / 0.1) ** (1 / 3)
    for prec in (rbe.FP64, rbe.FP32C):
        params = rbe.make_params(L, (3.0 / r) ** 2, r, r, 20, prec=prec, terms=rbe.TERM_LJ | rbe.TERM_COUL_REAL)
        ctx, st = rbe.Context(params, n), random_state(n, L, charged=0.1)
        t[prec] = best_us(lambda: ctx.energy(st))
        ctx.close()
    print(f"energy of {n}, {m} in the cutoff: {t}")
    assert t[rbe.FP32C] < 1.1 * t[rbe.FP64]


def test_energy_of_neutral_particles():
    """LJ pairs alone, 1,000 to a particle: their energies cost no more than their forces (1.18 of it from queues,
    0.90 summed as they are met)."""
    n, m = 300_000, 1_000
    r, L = (m / (4.0 / 3.0 * np.pi * 0.1)) ** (1 / 3), (n / 0.1) ** (1 / 3)
    ctx = rbe.Context(rbe.make_params(L, (3.0 / r) ** 2, r, r, 20, terms=rbe.TERM_LJ), n)
    st = random_state(n, L, charged=0.0)
    t = [best_us(lambda: f(st), reps=5) for f in (ctx.energy, ctx.forces)]
    ctx.close()
    print(f"LJ of {n}, {m} in the cutoff: energy, forces {t}")
    assert t[0] < 1.04 * t[1]


@pytest.mark.parametrize("n", [200_000, 700_000])
def test_random_batch_list_of_neighbouring_densities(n):
    """52 particles within r_coul on average against 45, on either side of the line between wide and narrow shells."""
    t, L = {}, (n / 0.1) ** (1 / 3)
    for m in (45, 52):
        r = (m / (4.0 / 3.0 * np.pi * 0.1)) ** (1 / 3)
        params = rbe.make_params(L, (3.0 / r) ** 2, r, 0.5 * r, 20, r_core=0.5 * r, p_shell=20,
                                 terms=rbe.TERM_LJ | rbe.TERM_COUL_REAL)
        ctx, st = rbe.Context(params, n), random_state(n, L)
        t[m] = best_us(lambda: ctx.forces(st), reps=10)
        ctx.close()
    print(f"batch list of {n}: {t}")
    assert t[52] < 1.16 * t[45]
