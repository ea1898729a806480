"""Performance cases of the SAIL annealing library: what its users have it do,
through the public binding, over the sizes, precisions and options in use.

Every case anneals seeded synthetic data (truncated Lorentzians, noise
proportional to the signal, the grids of the repository's workloads).  The
kinds:

  step    one sweep of a small population and its residues: the smallest call,
          as a program makes it that steers the temperature itself
  solve   a whole short anneal of one small problem, from fresh walkers to the
          averaged spectrum
  block   the next block of a running anneal (sweeps, resync, branching) and
          the read-out a program makes after each block
  batch   one round of many problems of mixed sizes sharing the device
  served  a burst of jobs handed to a server and waited for
  readout the averaged spectrum, the residues and their histogram of a
          population at rest: what a monitor reads between blocks

FP32 cases run the hot part of a schedule; there both precisions take the same
decisions, so their spectra can be compared value by value.
"""
import math

import numpy as np

from paper_1609_07936_amd import sail as S
from paper_1609_07936_amd import workloads as W

PRECISION = {"fp64": S.SAIL_FP64, "fp32": S.SAIL_FP32}


def _case(kind, **kw):
    c = dict(kind=kind, precision="fp64", n_omega=512, n_tau=128, n_walkers=16384, omega_max=20.0, tau_lo=0.02,
             tau_hi=3.0, weighted=True, mode="point", tile=0, n_T=20000, t_hi=1e3, t_lo=1e-2, sweeps=100,
             branch_every=100, resync_every=100, walk_len=0, smooth=0.0, adaptive=False, self_cool=False)
    c.update(kw)
    return c


def _band(**kw):
    """The paper's clipped Lorentzian band under its own protocol."""
    return _case("block", omega_max=3.5, tau_lo=0.0, tau_hi=6.3, weighted=False, self_cool=True, adaptive=True,
                 smooth=0.01, **kw)


def listed():
    return [
        # one sweep of the small reference problem: launch and chain latency
        _case("step", name="step_64x32_fp64", n_omega=64, n_tau=32, n_walkers=64, omega_max=10.0, tau_lo=0.05,
              tau_hi=1.6, n_T=2000, t_hi=1e2, t_lo=1e-3, sweeps=1),
        # the small reference problem solved outright, two branching events
        _case("solve", name="solve_64x32_fp64", n_omega=64, n_tau=32, n_walkers=64, omega_max=10.0, tau_lo=0.05,
              tau_hi=1.6, n_T=200, t_hi=1e2, t_lo=1e-3, sweeps=200),
        # the production anneal, block by block, in both precisions
        _case("block", name="block_512x128x16384_fp64"),
        _case("block", name="block_512x128x16384_fp32", precision="fp32", resync_every=50),
        # the paper's own problem and protocol, alone on the device
        _band(name="block_band_1000x64x1500_fp64", n_omega=1000, n_tau=64, n_walkers=1500, tile=4),
        # a user's odd grid: unweighted residue, exact bin integrals
        _case("block", name="block_301x77x3001_fp64", n_omega=301, n_tau=77, n_walkers=3001, omega_max=12.0,
              weighted=False, mode="bin_exact", n_T=2000, sweeps=50, branch_every=50, resync_every=25),
        # index selection by walks (proposals follow the spectrum)
        _case("block", name="block_walk_256x64x1024_fp64", n_omega=256, n_tau=64, n_walkers=1024, walk_len=4,
              n_T=2000, sweeps=20, branch_every=20, resync_every=20),
        # many users' problems at once: one shared round
        _case("batch", name="batch_64jobs_fp32", jobs=64, mix=1000, precision="fp32", n_T=1000, sweeps=50,
              resync_every=50, tile=16),
        _case("batch", name="batch_24jobs_fp64", jobs=24, mix=2000, n_T=1000, sweeps=50, resync_every=50, tile=16),
        # a burst of short jobs into the served loop
        _case("served", name="served_16jobs_fp32", jobs=16, mix=3000, precision="fp32", n_T=50, t_lo=1.0, sweeps=50,
              branch_every=50, resync_every=50, tile=16),
        # monitoring the production population
        _case("readout", name="readout_512x128x16384_fp64", sweeps=1),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "solve", "block", "block", "block32", "band", "walk", "batch", "batch32", "served",
                       "readout"])
    grid = dict(n_omega=_log_int(rng, 48, 900), n_tau=_log_int(rng, 24, 256), omega_max=rng.uniform(8.0, 20.0),
                tau_hi=rng.uniform(1.5, 3.0))
    small = dict(n_omega=_log_int(rng, 32, 128), n_tau=_log_int(rng, 16, 48), n_walkers=_log_int(rng, 32, 300),
                 omega_max=rng.uniform(6.0, 12.0), tau_lo=0.05, tau_hi=rng.uniform(1.0, 2.0), t_hi=1e2, t_lo=1e-3)
    if kind == "step":
        return _case("step", n_T=2000, sweeps=1, **small)
    if kind == "solve":
        n = rng.choice([100, 200, 300])
        return _case("solve", n_T=n, sweeps=n, **small)
    if kind in ("block", "block32"):
        f32 = kind == "block32"
        no = grid["n_omega"]
        # walkers over the whole range, kept inside the cost of the production block
        nw = min(_log_int(rng, 300, 16384), int(16384 * 512 / no))
        every = rng.choice([25, 50])
        return _case("block", precision="fp32" if f32 else "fp64", n_walkers=nw, sweeps=50, branch_every=50,
                     resync_every=every, weighted=f32 or rng.random() < 0.7,
                     mode=rng.choice(["point", "bin_exact"]), **grid)
    if kind == "band":
        return _band(n_omega=rng.randint(400, 1000), n_tau=rng.randint(33, 64), n_walkers=rng.randint(700, 1500),
                     tile=rng.choice([4, 8]), sweeps=50, branch_every=50, resync_every=50)
    if kind == "walk":
        return _case("block", n_omega=_log_int(rng, 96, 400), n_tau=_log_int(rng, 24, 128),
                     n_walkers=_log_int(rng, 200, 1500), walk_len=rng.randint(1, 6), n_T=2000, sweeps=20,
                     branch_every=20, resync_every=20)
    if kind in ("batch", "batch32"):
        f32 = kind == "batch32"
        return _case("batch", precision="fp32" if f32 else "fp64", jobs=rng.randint(6, 64 if f32 else 24),
                     mix=rng.randrange(10 ** 6), n_T=1000, sweeps=50, resync_every=rng.choice([25, 50]),
                     tile=rng.choice([8, 16]) if not f32 else 16)
    if kind == "served":
        return _case("served", precision=rng.choice(["fp32", "fp64"]), jobs=rng.randint(4, 16),
                     mix=rng.randrange(10 ** 6), n_T=50, t_lo=1.0, sweeps=50, branch_every=50, resync_every=50,
                     tile=16)
    return _case("readout", n_walkers=_log_int(rng, 1024, 16384), sweeps=1, **grid)


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _data(case, rng):
    """omega, tau, F, sigma, m0, m1 of a seeded target on the case's grid."""
    omega_max = case["omega_max"]
    if case["self_cool"]:
        c = rng.uniform(0.9, 1.1)
        target = W.Target([c, c + 1.0], [1.0, 1.0], [1.0, 1.0], omega_max, lo=0.5, hi=2.5)
    else:
        n_peaks = int(rng.integers(2, 4))
        target = W.Target(rng.uniform(0.5, 0.4 * omega_max, n_peaks), rng.uniform(0.05, 1.0, n_peaks),
                          0.1 + rng.dirichlet(np.ones(n_peaks)), omega_max)
    tau = W.uniform_tau(case["tau_lo"], case["tau_hi"], case["n_tau"])
    F, m0, m1 = W.transform_quadrature(target, tau, 4000)
    sigma = 10.0 ** rng.uniform(-5.0, -3.5) * F
    F = F + sigma * rng.standard_normal(F.size)
    return W.bin_centres(omega_max, case["n_omega"]), tau, F, sigma if case["weighted"] else None, m0, m1


def _schedule(case):
    T = W.geometric_schedule(case["t_hi"], case["t_lo"], case["n_T"])
    return S.Schedule(T, branch_every=case["branch_every"], resync_every=case["resync_every"],
                      walk_len=case["walk_len"], smooth=case["smooth"], adaptive=int(case["adaptive"]),
                      self_cool=int(case["self_cool"]), boil_blocks=20, cool_blocks=100)


def _mix(case):
    """The sizes of a batch's or a burst's jobs (bins, times, walkers)."""
    rng = np.random.default_rng(case["mix"])
    walkers = [256, 1024] if case["kind"] == "served" else [256, 1024, 4096]
    return [dict(case, n_omega=int(rng.choice([128, 256, 512, 1024])), n_tau=int(rng.choice([32, 64, 128, 256])),
                 n_walkers=int(rng.choice(walkers))) for _ in range(case["jobs"])]


def _problem(case, rng):
    omega, tau, F, sigma, m0, m1 = _data(case, rng)
    p = S.Problem(omega, tau, F, sigma, m0, m1,
                  S.SAIL_K_BIN_EXACT if case["mode"] == "bin_exact" else S.SAIL_K_POINT)
    p.set_tau_per_lane(case["tile"])
    return p


def prepare(case, seed):
    rng = np.random.default_rng(seed)
    precision = PRECISION[case["precision"]]
    state = {"case": case, "seed": int(seed), "sched": _schedule(case), "k": 0}
    if case["kind"] == "served":
        state["server"] = S.Server(2 << 30, 64)
        state["jobs"] = [(_data(j, rng), j["n_walkers"], int(seed) + i) for i, j in enumerate(_mix(case))]
        return state
    if case["kind"] == "batch":
        state["problems"] = [_problem(j, rng) for j in _mix(case)]
        for i, (p, j) in enumerate(zip(state["problems"], _mix(case))):
            p.init_walkers(j["n_walkers"], int(seed) + i, precision)
        state["batch"] = S.Batch(state["problems"])
        return state
    state["problem"] = p = _problem(case, rng)
    if case["kind"] != "solve":
        p.init_walkers(case["n_walkers"], int(seed), precision)
    if case["kind"] == "readout":
        p.run(state["sched"], 0, case["sweeps"])
    return state


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
def _next(state):
    """First sweep of the next stretch of the schedule (from its start again
    after its end)."""
    n, k = state["case"]["sweeps"], state["k"]
    if k + n > state["case"]["n_T"]:
        k = 0
    state["k"] = k + n
    return k


def run(state):
    case, sched = state["case"], state["sched"]
    kind, n = case["kind"], case["sweeps"]
    if kind == "served":
        srv, prec = state["server"], PRECISION[case["precision"]]
        ids = [srv.submit(*data, n_walkers, seed, sched, precision=prec, tau_per_lane=case["tile"])
               for data, n_walkers, seed in state["jobs"]]
        res = [srv.wait(i) for i in ids]
        return {"spectra": np.concatenate([r["mean_spectrum"] for r in res]),
                "chi2_min": np.array([r["chi2_min"] for r in res]),
                "chi2_median": np.array([r["chi2_median"] for r in res]),
                "chi2_unit": np.array([r["chi2_unit"] for r in res])}
    if kind == "batch":
        state["batch"].run(sched, _next(state), n)
        return {"spectra": np.concatenate([p.read_spectrum() for p in state["problems"]]),
                "chi2": np.concatenate([p.read_chi2() for p in state["problems"]])}
    p = state["problem"]
    if kind == "readout":
        return {"spectrum": p.read_spectrum(), "chi2": p.read_chi2(), "hist": p.read_chi2_hist(64)}
    if kind == "solve":
        p.init_walkers(case["n_walkers"], state["seed"], PRECISION[case["precision"]])
        p.run(sched, 0, n)
        ev = p.read_events(n // case["branch_every"])
        return {"spectrum": p.read_spectrum(), "chi2": p.read_chi2(), "zeros": ev["z"], **p.read_state()}
    p.run(sched, _next(state), n)
    out = {"chi2": p.read_chi2()}
    if kind == "block":
        out["spectrum"] = p.read_spectrum()
    return out


def work(case):
    """Per proposal the two coefficients it draws and the 8 flops per time
    point of its residue change (two columns scaled and added, the change
    weighted against the residual and itself); per read-out the spectra once."""
    if case["kind"] in ("batch", "served"):
        ws = [work(dict(j, kind="block")) for j in _mix(case)]
        return {k: sum(w[k] for w in ws) for k in ("bytes", "flops")}
    state = 8.0 * case["n_walkers"] * (case["n_omega"] + 1)
    if case["kind"] == "readout":
        return {"bytes": state, "flops": 2.0 * case["n_walkers"] * case["n_omega"]}
    proposals = float(case["n_walkers"]) * case["n_omega"] * case["sweeps"]
    return {"bytes": 2.0 * state, "flops": 8.0 * case["n_tau"] * proposals}


# ---------------------------------------------------------------------------
# the same anneal in plain numpy, 64 bits
# ---------------------------------------------------------------------------
def _philox(c0, c1, c2, c3, key):
    """Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11) on arrays of counters."""
    m32 = np.uint64(0xFFFFFFFF)
    c = [np.asarray(v, dtype=np.uint64) for v in (c0, c1, c2, c3)]
    k0, k1 = key & 0xFFFFFFFF, key >> 32
    for _ in range(10):
        p0, p1 = np.uint64(0xD2511F53) * c[0], np.uint64(0xCD9E8D57) * c[2]
        c = [(p1 >> np.uint64(32)) ^ c[1] ^ np.uint64(k0), p1 & m32,
             (p0 >> np.uint64(32)) ^ c[3] ^ np.uint64(k1), p0 & m32]
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return c


def _tilted(omega, A, B):
    """a_j ~ e^{-lambda omega_j} with sum a = A and sum omega a = B."""
    mu = B / A

    def shape(lam):
        e = np.exp(-lam * (omega - (omega[0] if lam > 0 else omega[-1])))
        return e / e.sum()

    lo, hi = -1.0, 1.0
    while shape(lo) @ omega < mu:
        lo *= 2.0
    while shape(hi) @ omega > mu:
        hi *= 2.0
    for _ in range(200):
        mid = 0.5 * (lo + hi)
        lo, hi = (mid, hi) if shape(mid) @ omega > mu else (lo, mid)
    a = A * shape(0.5 * (lo + hi))
    s0, s1, s2 = a.sum(), a @ omega, a @ omega ** 2
    d0, d1 = np.linalg.solve([[s0, s1], [s1, s2]], [A - s0, B - s1])
    return a + a * (d0 + d1 * omega)


def exact(case, seed):
    """Sweeps of uniform selection up to the first resync, walker by walker in
    FP64 numpy; None for stretches with resyncs or branching events, and for
    reads of populations too large to follow this way."""
    if case["kind"] != "step" or case["sweeps"] >= case["resync_every"]:
        return None
    omega, tau, F, sigma, m0, m1 = _data(case, np.random.default_rng(seed))
    n, No = case["n_walkers"], omega.size
    dw = omega[1] - omega[0]
    A, B = m0 / dw, m1 / dw
    K = np.exp(-np.outer(omega, tau)) * dw / (2.0 * np.pi)
    w = np.ones_like(F) if sigma is None else 1.0 / sigma ** 2
    a = np.tile(_tilted(omega, A, B), (n, 1))
    R = a @ K - F
    chi2 = (w * R * R).sum(1)
    T = W.geometric_schedule(case["t_hi"], case["t_lo"], case["n_T"]) * chi2[0]
    lane = np.arange(n)
    rate = np.ones(n)
    for k in range(case["sweeps"]):
        y = np.minimum(rate, 1.0) ** 2
        taken = np.zeros(n)
        for q in range(No):
            x = _philox(np.full(n, q), np.full(n, k), lane, np.zeros(n), int(seed))
            u = [(v.astype(np.float64) + 0.5) * 2.0 ** -32 for v in x]
            p, s = ((v * np.uint64(No)) >> np.uint64(32) for v in x[:2])
            p, s = p.astype(np.int64), s.astype(np.int64)
            r = 1.0 - y * 0.1 * (2.0 * u[2] - 1.0)
            gap = np.where(p == s, 1.0, omega[p] - omega[s])
            dp, ds = (1.0 - r) * (B - A * omega[s]) / gap, -(1.0 - r) * (B - A * omega[p]) / gap
            ap, as_ = r * a[lane, p] + dp, r * a[lane, s] + ds
            dF = (r - 1.0)[:, None] * (R + F) + dp[:, None] * K[p] + ds[:, None] * K[s]
            d = (w * dF * (2.0 * R + dF)).sum(1)
            ok = (p != s) & (ap >= 0.0) & (as_ >= 0.0) & (d < -T[k] * np.log(u[3]))
            g = np.where(ok, r, 1.0)
            a *= g[:, None]
            a[lane[ok], p[ok]], a[lane[ok], s[ok]] = ap[ok], as_[ok]
            R[ok] += dF[ok]
            chi2 = chi2 + np.where(ok, d, 0.0)
            taken += ok
        rate = 0.9 * rate + 0.1 * taken / No
    return {"chi2": (w * (a @ K - F) ** 2).sum(1)}
