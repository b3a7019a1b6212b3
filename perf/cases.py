"""Performance cases of the random batch Ewald force and its dynamics.

Every case is a call that a user's simulation makes through the public
binding: one force evaluation, a run of velocity-Verlet or Nose-Hoover steps,
an energy diagnostic, a batch of replicas. The physics are the workloads of
this repository's benchmark (point charges with 12-6 LJ cores, reduced
units): plain ions, the random batch list electrolyte, the ghost-shell
subdomain, replicas, and the dilute LJ electrolyte run under NVT.

listed()  the fixed cases         draw(rng)  one more case of the same ranges
prepare() inputs and the context  run()      one pass, and its outputs
work()    bytes and flops of a pass that cannot be avoided
exact()   the same outputs in 64 bits, in plain torch and numpy
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2609_02694_amd as rbe

# Physics of the workloads: number density, share of charged particles,
# splitting parameter, cutoffs, batch list, step. h, k: the edge of the y/z
# cells and the x cells per edge that the autotuner picks (grid "tuned";
# grid "default" leaves the choice to the library).
PHYSICS = {
    "ions": dict(density=3000 / 30.0**3, charged=1.0, alpha=0.3, r_coul=8.0, r_lj=2.5, r_core=0.0, p_shell=0,
                 dt=0.002, ghost=0.0, h=4.0, k=6),
    "electrolyte": dict(density=0.8, charged=0.25, alpha=0.35, r_coul=6.0, r_lj=2.5, r_core=3.0, p_shell=20,
                        dt=0.002, ghost=0.0, h=3.0, k=6),
    "replica": dict(density=0.5, charged=0.5, alpha=0.3, r_coul=6.0, r_lj=2.5, r_core=0.0, p_shell=0,
                    dt=0.002, ghost=0.0, h=2.5, k=3),
    "subdomain": dict(density=0.8, charged=0.10, alpha=0.35, r_coul=6.0, r_lj=2.5, r_core=0.0, p_shell=0,
                      dt=0.002, ghost=6.0, h=2.5, k=4),
    "ljelectrolyte": dict(density=200_000 / 271.0**3, charged=1.0, alpha=(3.0 / 8.0) ** 2, r_coul=8.0, r_lj=8.0,
                          r_core=4.0, p_shell=30, dt=0.001, ghost=0.0, h=8.2, k=4),
}
KT, TAU = 1.0, 0.1  # Nose-Hoover target and relaxation time of the NVT cases


def _case(name, call, physics, n, prec, P, steps=1, grid="default", nvt=False, replicas=1, ewald=False):
    c = dict(call=call, physics=physics, n=n, prec=prec, P=P, steps=steps, grid=grid, nvt=nvt, replicas=replicas,
             ewald=ewald)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest call: one force evaluation of a few thousand ions, as a
        # driver with an integrator of its own makes it every step
        _case("forces_ions_3k_fp64", "forces", "ions", 3000, "fp64", 100),
        # the same without a context, under capture or where nothing may allocate; an odd size
        _case("noalloc_replica_10k_fp64", "noalloc", "replica", 10_007, "fp64", 128),
        # a small system's dynamics on its own: launches and latency
        _case("step_replica_2k_fp32c", "step", "replica", 2001, "fp32c", 100, steps=20, grid="tuned", nvt=True),
        # plain Ewald dynamics through the library (every lattice mode, no batch
        # list): the reference run that the random batch estimates are checked with
        _case("step_ewald_4k_fp64", "step", "ljelectrolyte", 4000, "fp64", 0, steps=2, nvt=True, ewald=True),
        # the energy and pressure report of a production run
        _case("energy_electrolyte_200k_fp64", "energy", "electrolyte", 200_001, "fp64", 200),
        # the LJ electrolyte of the method's accuracy and timing study, NVT
        _case("step_ljelectrolyte_200k_fp64", "step", "ljelectrolyte", 200_000, "fp64", 200, steps=5, grid="tuned",
              nvt=True),
        # dense electrolyte with the random batch list
        _case("step_electrolyte_1m_fp64", "step", "electrolyte", 1_000_000, "fp64", 200, steps=4, grid="tuned"),
        # many independent replicas of uneven size, both precisions
        _case("batch_replica_256_fp32c", "step", "replica", 3_400_000, "fp32c", 100, steps=5, grid="tuned",
              replicas=256),
        _case("batch_replica_24_fp64", "step", "replica", 150_000, "fp64", 100, steps=5, grid="default",
              replicas=24),
        # ions only, single precision with compensation
        _case("step_ions_8m_fp32c", "step", "ions", 8_000_000, "fp32c", 500, steps=2, grid="tuned"),
        # one device's subdomain with its ghost shell: double precision, and
        # the largest system in the compensated form
        _case("step_subdomain_8m_fp64", "step", "subdomain", 8_000_001, "fp64", 1000, steps=2, grid="tuned"),
        _case("step_subdomain_64m_fp32c", "step", "subdomain", 64_000_000, "fp32c", 1000, steps=2, grid="tuned"),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    call = rng.choice(["forces", "step", "step", "step", "batch", "energy", "noalloc", "ewald"])
    prec = rng.choice(["fp64", "fp64", "fp32c"])
    P = _log_uniform(rng, 20, 1000)
    grid = rng.choice(["default", "tuned"])
    if call == "ewald":
        return _case(None, "step", "ljelectrolyte", _log_uniform(rng, 500, 6000), prec, 0, steps=2, nvt=True,
                     ewald=True)
    if call == "batch":
        replicas = _log_uniform(rng, 2, 256)
        n = replicas * _log_uniform(rng, 1200, 12_000)
        return _case(None, "step", "replica", n + rng.randrange(64), prec, _log_uniform(rng, 20, 200), steps=5,
                     grid=grid, replicas=replicas)
    if call == "noalloc":
        physics = rng.choice(["ions", "replica", "electrolyte"])
        return _case(None, call, physics, _log_uniform(rng, 1500, 32_768), prec, P)
    physics = rng.choice(list(PHYSICS))
    if call == "energy":
        return _case(None, call, physics, _log_uniform(rng, 1500, 500_000), prec, P, grid=grid)
    n = _log_uniform(rng, 1500, 3_000_000)
    if call == "forces":
        return _case(None, call, physics, n, prec, P, grid=grid)
    steps = 20 if n < 20_000 else 5 if n < 300_000 else 2
    # a lone small system is run under the thermostat, as sampled forces heat it
    nvt = n < 100_000 or physics == "ljelectrolyte" or rng.random() < 0.3
    return _case(None, call, physics, n, prec, P, steps=steps, grid=grid, nvt=nvt)


# ---------------------------------------------------------------------------
# systems
# ---------------------------------------------------------------------------
def _sizes(case):
    """Particles per replica: log-uniform between 1,000 and about sixty times that, scaled to the total."""
    r, n = case["replicas"], case["n"]
    if r == 1:
        return [n]
    g = np.random.default_rng(1004)
    u = np.exp(g.uniform(0.0, math.log(60.0), r))
    spare = n - 1000 * r
    share = np.floor(spare * u / u.sum()).astype(np.int64)
    return [int(v) for v in 1000 + share]


def _kmax(ph):
    # every mode whose Gaussian factor is at least 1e-7
    return math.sqrt(4.0 * ph["alpha"] * math.log(1e7))


def _params(case, n, seed):
    ph = PHYSICS[case["physics"]]
    L = (n / ph["density"]) ** (1.0 / 3.0)
    nc = (0, 0, 0)
    if case["grid"] == "tuned":
        c = max(1, int(L // ph["h"]))
        nc = (c * ph["k"], c, c)
    nvt = case["nvt"]
    make = lambda P: rbe.make_params(  # noqa: E731
        L, ph["alpha"], ph["r_coul"], ph["r_lj"], P, 0.0 if case["ewald"] else ph["r_core"],
        0 if case["ewald"] else ph["p_shell"], prec=rbe.FP64 if case["prec"] == "fp64" else rbe.FP32C, ncell=nc,
        dt=ph["dt"], ghost_width=ph["ghost"], seed=seed, nvt_kT=KT if nvt else 0.0, nvt_tau=TAU if nvt else 0.0)
    if case["ewald"]:
        m, w = rbe.lattice_modes(make(1), _kmax(ph))
        return make(m.shape[1]), L, (m, w)
    return make(case["P"]), L, None


def _system(case, n, L, gen, device):
    """A disordered system: randomly occupied lattice sites, each displaced at
    random while no two particles come closer than 0.8, random charges, and
    velocities at kT = 1. Particles come in random order."""
    ph = PHYSICS[case["physics"]]
    side = math.ceil(n ** (1.0 / 3.0) - 1e-9)
    a = L / side
    site = torch.randperm(side**3, generator=gen, device=device)[:n]
    jitter = max(0.02, 0.5 * (a - 0.8))
    r = {}
    for name, cell in (("x", site % side), ("y", (site // side) % side), ("z", site // (side * side))):
        u = torch.rand(n, generator=gen, device=device, dtype=torch.float64)
        u.mul_(2.0).sub_(1.0).mul_(jitter).add_((cell.to(torch.float64) + 0.5) * a)
        r[name] = torch.remainder(u, L)
    del site
    for name in ("vx", "vy", "vz"):
        r[name] = torch.randn(n, generator=gen, device=device, dtype=torch.float64)
    half = int(n * ph["charged"]) // 2
    q = torch.zeros(n, device=device, dtype=torch.float64)
    q[:half] = 1.0
    q[half: 2 * half] = -1.0
    r["q"] = q[torch.randperm(n, generator=gen, device=device)]
    r["id"] = torch.arange(n, device=device, dtype=torch.int32)
    return r


KEYS = ("x", "y", "z", "vx", "vy", "vz", "q", "id")


def _inputs(case, seed, device):
    """Parameters of every replica, their box edges, offsets, the state arrays and the mode table of an Ewald run."""
    gen = torch.Generator(device=device).manual_seed(int(seed))
    sizes = _sizes(case)
    params, edges, parts, modes = [], [], [], None
    for k, n in enumerate(sizes):
        p, L, modes = _params(case, n, (int(seed) << 12) + k)
        params.append(p)
        edges.append(L)
        parts.append(_system(case, n, L, gen, device))
    cat = parts[0] if len(parts) == 1 else {k: torch.cat([s[k] for s in parts]) for k in KEYS}
    off = [0]
    for n in sizes:
        off.append(off[-1] + n)
    return params, edges, off, cat, modes


def prepare(case, seed):
    params, _, off, cat, modes = _inputs(case, seed, "cuda")
    n = off[-1]
    zero = lambda: torch.zeros(n, dtype=torch.float64, device="cuda")  # noqa: E731
    nh = torch.zeros(2, dtype=torch.float64, device="cuda") if case["nvt"] else None
    st = rbe.Particles(cat["x"], cat["y"], cat["z"], cat["vx"], cat["vy"], cat["vz"], zero(), zero(), zero(), cat["q"],
                       cat["id"], nh)
    state = dict(case=case, st=st, params=params[0], ev=0)
    if case["call"] == "noalloc":
        m, w = rbe.sample_k(params[0], 0)
        state["m"] = torch.as_tensor(m.ravel()).cuda()
        state["w"] = torch.as_tensor(w).cuda()
        return state
    if case["replicas"] > 1:
        ctx = rbe.Context.batch(params, off)
    else:
        ctx = rbe.Context(params[0], n)
    if modes is not None:
        ctx.set_modes(torch.as_tensor(modes[0].ravel()).cuda(), torch.as_tensor(modes[1]).cuda())
    state["ctx"] = ctx
    if case["call"] == "step":
        # a step starts from the force of the current positions
        ctx.forces(st, ev=0)
        ctx.sync_check()
        state["ev"] = 1
    return state


def run(state):
    case, st = state["case"], state["st"]
    ev = state["ev"]
    if case["call"] == "noalloc":
        rbe.forces_noalloc(state["params"], st, state["m"], state["w"], ev)
        return {"fx": st.fx, "fy": st.fy, "fz": st.fz}
    ctx = state["ctx"]
    if case["call"] == "forces":
        state["ev"] = ev + 1
        ctx.forces(st, ev=ev)
        return {"fx": st.fx, "fy": st.fy, "fz": st.fz}
    if case["call"] == "energy":
        state["ev"] = ev + 1
        return ctx.energy(st, ev=ev)
    state["ev"] = ev + case["steps"]
    ctx.step(st, case["steps"], ev)
    out = {k: getattr(st, k) for k in KEYS + ("fx", "fy", "fz")}
    if st.nh is not None:
        out["nh"] = st.nh
    return out


# ---------------------------------------------------------------------------
# work of one pass
# ---------------------------------------------------------------------------
def _mode_count(case):
    if not case["ewald"]:
        return case["P"]
    ph = PHYSICS[case["physics"]]
    V = case["n"] / ph["density"]
    return 0.5 * (4.0 / 3.0) * math.pi * _kmax(ph) ** 3 * V / (2.0 * math.pi) ** 3


def work(case):
    """Flops of the pair terms inside the cutoffs (27 a Coulomb term, 22 an LJ
    term) and of the Fourier terms (13 a particle and mode for the structure
    factors, 18 for the forces), and the bytes of the state, in and out once
    per step."""
    ph = PHYSICS[case["physics"]]
    n, rho = case["n"], PHYSICS[case["physics"]]["density"]
    nq = n * ph["charged"]
    ball = lambda r: 4.0 / 3.0 * math.pi * r**3  # noqa: E731
    if ph["r_core"] > 0 and not case["ewald"] and case["call"] != "energy":
        coul = nq * (rho * ph["charged"] * ball(ph["r_core"]) + ph["p_shell"] * ph["charged"])
        lj = n * rho * ball(min(ph["r_lj"], ph["r_core"])) + (nq * ph["p_shell"] if ph["r_lj"] > ph["r_core"] else 0)
    else:
        coul = nq * rho * ph["charged"] * ball(ph["r_coul"])
        lj = n * rho * ball(ph["r_lj"])
    P = _mode_count(case)
    if case["call"] == "energy":
        # each pair once
        return {"bytes": n * 56.0 + 64.0, "flops": 0.5 * (27.0 * coul + 22.0 * lj) + 13.0 * nq * P}
    flops = 27.0 * coul + 22.0 * lj + 31.0 * nq * P
    if case["call"] == "step":
        return {"bytes": case["steps"] * n * 2.0 * 84.0, "flops": case["steps"] * flops}
    return {"bytes": n * (36.0 + 24.0), "flops": flops}


# ---------------------------------------------------------------------------
# the same results in 64 bits, in plain torch and numpy
# ---------------------------------------------------------------------------
_GAMMA = 0x9E3779B97F4A7C15


def _mix64(z):
    z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
    z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
    return z ^ (z >> np.uint64(31))


def _stream(s, k):
    """Output k (0-based) of the SplitMix64 stream seeded by s."""
    with np.errstate(over="ignore"):
        return _mix64(np.uint64(s) + (np.asarray(k, np.uint64) + np.uint64(1)) * np.uint64(_GAMMA))


def _sample(seed, ev, L, alpha, P):
    """The importance sample of lattice modes: per-axis inverse CDFs of exp(-(pi m / L)^2 / alpha), m = 0 rejected."""
    M = math.ceil(L * math.sqrt(40.0 * alpha) / math.pi)
    a = np.array([math.pi * float(i - M) / L for i in range(2 * M + 1)])
    acc = np.cumsum(np.array([math.exp(-(v * v) / alpha) for v in a]))
    S = acc[-1] ** 3 - 1.0
    cdf = acc / acc[-1]
    kl = _stream(_stream(seed ^ 0x4B4D4F4445534554, ev), np.arange(P, dtype=np.uint64))
    m = np.zeros((P, 3), np.int64)
    todo = np.arange(P)
    t = 0
    while len(todo):
        u = np.stack([_output(kl[todo], 3 * t + d) for d in range(3)], axis=1)
        m[todo] = np.searchsorted(cdf, (u >> np.uint64(11)).astype(np.float64) * 2.0**-53, side="right") - M
        todo = todo[(m[todo] == 0).all(axis=1)]
        t += 1
    k2 = ((2.0 * math.pi * m / L) ** 2).sum(axis=1)
    return m, (S / P) * 4.0 * math.pi / (L**3 * k2)


def _output(keys, k):
    """Output k of the streams seeded by keys."""
    with np.errstate(over="ignore"):
        return _mix64(keys + np.uint64(k + 1) * np.uint64(_GAMMA))


def _lattice(L, alpha, kmax):
    """Half-space lattice modes up to kmax with the Ewald weights (each for itself and its negative)."""
    M = int(math.floor(kmax * L / (2.0 * math.pi)))
    g = np.arange(-M, M + 1)
    mx, my, mz = (v.ravel() for v in np.meshgrid(np.arange(0, M + 1), g, g, indexing="ij"))
    k2 = ((2.0 * math.pi / L) ** 2) * (mx * mx + my * my + mz * mz)
    keep = (k2 <= kmax * kmax) & ((mx > 0) | (my > 0) | ((my == 0) & (mz > 0)))
    m, k2 = np.stack([mx, my, mz], axis=1)[keep], k2[keep]
    return m, 8.0 * math.pi * np.exp(-k2 / (4.0 * alpha)) / (L**3 * k2)


def _mul32(a, b):
    return (a * b) & 0xFFFFFFFF


def _low32(x):
    x = x ^ (x >> 16)
    x = _mul32(x, 0x7FEB352D)
    x = x ^ (x >> 15)
    x = _mul32(x, 0x846CA68B)
    return x ^ (x >> 16)


class _Exact:
    """Force, energy and motion of one system, by all pairs."""

    def __init__(self, case, L, seed, modes):
        self.case, self.L, self.seed, self.modes = case, L, seed, modes
        self.ph = PHYSICS[case["physics"]]

    def _modes(self, ev, device):
        m, w = self.modes if self.modes is not None else _sample(self.seed, ev, self.L, self.ph["alpha"],
                                                                 self.case["P"])
        return (torch.as_tensor(np.ascontiguousarray(m), dtype=torch.float64, device=device),
                torch.as_tensor(np.ascontiguousarray(w), dtype=torch.float64, device=device))

    def fourier(self, s, ev):
        """Forces on the charged particles, and w |rho|^2 / 2 summed with its virial weight."""
        dev = s["x"].device
        charged = torch.nonzero(s["q"] != 0).ravel()
        f = torch.zeros(len(s["x"]), 3, dtype=torch.float64, device=dev)
        if not len(charged):
            return f, 0.0, 0.0
        r = torch.stack([s["x"], s["y"], s["z"]], 1)[charged]
        q = s["q"][charged]
        m, w = self._modes(ev, dev)
        g = torch.zeros_like(r)
        u = v = 0.0
        step = max(1, int(3e7 // len(charged)))
        for a in range(0, len(w), step):
            mm, ww = m[a:a + step], w[a:a + step]
            # one axis at a time and whole turns taken out: the phase stays accurate
            t = sum(torch.frac(r[:, None, d] / self.L * mm[None, :, d]) for d in range(3)) * (2.0 * math.pi)
            c, sn = torch.cos(t), torch.sin(t)
            re, im = q @ c, q @ sn
            h = c * (ww * im) - sn * (ww * re)
            g += h @ mm
            e = 0.5 * ww * (re * re + im * im)
            k2 = ((2.0 * math.pi / self.L) ** 2) * (mm * mm).sum(1)
            u += float(e.sum())
            v += float((e * (1.0 - k2 / (2.0 * self.ph["alpha"]))).sum())
        f[charged] = -q[:, None] * (2.0 * math.pi / self.L) * g
        return f, u, v

    def near(self, s, ev):
        """Near-field forces (with the random batch list where the case has
        one), and the pair energies and virials over the cutoffs."""
        ph, L = self.ph, self.L
        dev = s["x"].device
        r, q, ids = torch.stack([s["x"], s["y"], s["z"]], 1), s["q"], s["id"].to(torch.int64)
        n = len(q)
        energy = self.case["call"] == "energy"
        rbl = ph["r_core"] > 0 and not self.case["ewald"] and not energy
        rc2, rl2, r02 = ph["r_coul"] ** 2, ph["r_lj"] ** 2, ph["r_core"] ** 2
        sa = math.sqrt(ph["alpha"])
        if rbl:
            h = _stream(_stream(self.seed ^ 0x52424C5348454C4C, ev), ids.cpu().numpy().astype(np.uint64))
            ka = torch.as_tensor((h & np.uint64(0xFFFFFFFF)).astype(np.int64), device=dev)
            kb = torch.as_tensor((h >> np.uint64(32)).astype(np.int64), device=dev)
        f = torch.zeros(n, 3, dtype=torch.float64, device=dev)
        e = torch.zeros(4, dtype=torch.float64, device=dev)
        step = max(1, int(2e8 // n))
        reach = max(rc2, rl2)
        for a in range(0, n, step):
            b = min(n, a + step)
            r2 = torch.zeros(b - a, n, dtype=torch.float64, device=dev)
            for d in range(3):
                dd = r[a:b, None, d] - r[None, :, d]
                dd -= L * torch.round(dd / L)
                r2 += dd.square_()
            r2[torch.arange(b - a, device=dev), torch.arange(a, b, device=dev)] = math.inf
            i, j = torch.nonzero(r2 <= reach, as_tuple=True)
            rr = r2[i, j]
            del r2
            d3 = r[a + i] - r[j]
            d3 -= L * torch.round(d3 / L)
            qq = q[a + i] * q[j]
            rd = torch.sqrt(rr)
            er, ex = torch.erfc(sa * rd) / rd, torch.exp(-ph["alpha"] * rr)
            in_c, in_l = (rr <= rc2) & (qq != 0), rr <= rl2
            s6 = rr.pow(-3)
            coul = torch.where(in_c, qq * (er / rr + 2.0 * sa / math.sqrt(math.pi) * ex / rr), 0.0)
            lj = torch.where(in_l, 24.0 * (2.0 * s6 * s6 - s6) / rr, 0.0)
            if energy:
                e[0] += 0.5 * torch.where(in_c, qq * er, 0.0).sum()
                e[1] += 0.5 * torch.where(in_l, 4.0 * (s6 * s6 - s6), 0.0).sum()
                e[2] += 0.5 * (coul * rr).sum()
                e[3] += 0.5 * (lj * rr).sum()
                continue
            weight = torch.ones_like(rr)
            if rbl:
                shell = (rr > r02) & (rr <= rc2) & ((q[a + i] != 0) | (ph["r_lj"] > ph["r_core"]))
                weight = torch.where(rr <= r02, 1.0, 0.0)
                at = torch.nonzero(shell).ravel()
                si = i[at]
                key = _low32(_low32(ids[j[at]] ^ ka[a + si]) ^ kb[a + si])
                order = torch.argsort(key)
                order = order[torch.argsort(si[order], stable=True)]
                at, si = at[order], si[order]
                count = torch.bincount(si, minlength=b - a)
                first = torch.cumsum(count, 0) - count
                place = torch.arange(len(si), device=dev) - first[si]
                batch = torch.clamp(count, max=ph["p_shell"])
                sel = place < batch[si]
                weight[at[sel]] = (count[si] / batch[si].to(torch.float64))[sel]
            f.index_add_(0, a + i, ((coul + lj) * weight)[:, None] * d3)
        if rbl:
            f -= f.mean(0)
        return f, e

    def force(self, s, ev):
        near, _ = self.near(s, ev)
        return near + self.fourier(s, ev)[0]

    def energy(self, s, ev):
        _, e = self.near(s, ev)
        _, u, v = self.fourier(s, ev)
        self_u = math.sqrt(self.ph["alpha"] / math.pi) * float(s["q"].square().sum())
        kin = 0.5 * float(sum(s[k].square().sum() for k in ("vx", "vy", "vz")))
        return torch.tensor([float(e[0]), float(e[1]), u, self_u, kin, float(e[2]), float(e[3]), v],
                            dtype=torch.float64)

    def cells(self, s, nc):
        c = []
        for k, n in zip(("x", "y", "z"), nc):
            c.append(torch.clamp((s[k] * (n / self.L)).floor().to(torch.int64), max=n - 1))
        key = (s["q"] == 0).to(torch.int64) * (nc[0] * nc[1] * nc[2]) + (c[2] * nc[1] + c[1]) * nc[0] + c[0]
        return torch.argsort(key, stable=True)

    def steps(self, s, nc, nh):
        dt, h = self.ph["dt"], 0.5 * self.ph["dt"]
        n = len(s["x"])
        nf = 3.0 * n - 3.0
        f = self.force(s, 0)
        v = torch.stack([s["vx"], s["vy"], s["vz"]], 1)

        def half():
            Q = nf * KT * TAU * TAU
            K = 0.5 * float(v.square().sum())
            nh[0] += 0.25 * dt * ((2.0 * K - nf * KT) / Q)
            sc = math.exp(-0.5 * dt * nh[0])
            nh[1] += 0.5 * dt * nh[0]
            K *= sc * sc
            nh[0] += 0.25 * dt * ((2.0 * K - nf * KT) / Q)
            v.mul_(sc)

        for k in range(self.case["steps"]):
            if nh is not None:
                half()
            v += h * f
            for d, x in enumerate(("x", "y", "z")):
                s[x] = s[x] + dt * v[:, d]
                s[x] = s[x] - self.L * torch.floor(s[x] / self.L)
            o = self.cells(s, nc)
            s = {key: t[o] for key, t in s.items()}
            v = v[o]
            f = self.force(s, 1 + k)
            v += h * f
            if nh is not None:
                half()
        s["vx"], s["vy"], s["vz"] = v[:, 0].contiguous(), v[:, 1].contiguous(), v[:, 2].contiguous()
        s["fx"], s["fy"], s["fz"] = f[:, 0].contiguous(), f[:, 1].contiguous(), f[:, 2].contiguous()
        return s


def _grid(case, L):
    """Cells per axis (the library's default where the case asks for it)."""
    ph = PHYSICS[case["physics"]]
    if case["grid"] == "tuned":
        c = max(1, int(L // ph["h"]))
        return (c * ph["k"], c, c)
    c = max(1, int(math.floor(L / max(ph["r_lj"], 0.5 * ph["r_coul"]))))
    return (4 * c, c, c)


def exact(case, seed):
    ph = PHYSICS[case["physics"]]
    evals = 1 + case["steps"] if case["call"] == "step" else 1
    pairs = sum(float(n) * n for n in _sizes(case))
    terms = case["n"] * ph["charged"] * _mode_count(case)
    if evals * (pairs + 3.0 * terms) > 6e10:
        return None
    dev = "cuda"
    _, edges, off, cat, _ = _inputs(case, seed, dev)
    parts = []
    for k, L in enumerate(edges):
        s = {key: cat[key][off[k]: off[k + 1]] for key in KEYS}
        modes = _lattice(L, ph["alpha"], _kmax(ph)) if case["ewald"] else None
        E = _Exact(case, L, (int(seed) << 12) + k, modes)
        if case["call"] == "energy":
            return E.energy(s, 0)
        if case["call"] in ("forces", "noalloc"):
            f = E.force(s, 0)
            return {"fx": f[:, 0].contiguous(), "fy": f[:, 1].contiguous(), "fz": f[:, 2].contiguous()}
        nh = [0.0, 0.0] if case["nvt"] else None
        parts.append(E.steps(s, _grid(case, L), nh))
    out = {key: torch.cat([p[key] for p in parts]) for key in KEYS + ("fx", "fy", "fz")}
    if case["nvt"]:
        out["nh"] = torch.tensor(nh, dtype=torch.float64)
    return out
