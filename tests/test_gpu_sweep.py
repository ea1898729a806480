"""GPU: the sweep's launch plans and basis classes at their edges.

A problem swept alone (its own plan), under a trace window (plain four-lane
plan) and in a batch (split or walk plan of the shared launch) has the same
bits, whatever the plan: compared with array_equal.  Problems whose weights
spread the columns over more dimensions (the wider classes, and the general
one of any number) are compared with the oracle, to the parity tests' bars.
"""
import dataclasses
import sys

import numpy as np
import pytest

from paper_1609_07936_amd import workloads as W
from test_gpu_parity import S, _anneal_lockstep  # noqa: F401 (the fixture)

pytestmark = pytest.mark.gpu


def _workload(n_omega, n_tau, n_walkers, n_sweeps, spread=0.0):
    """A two-peak target; spread > 0 weights the times so that the columns
    sqrt(w_i) e^{-omega_j tau_i} become Gaussians along tau, whose rank grows
    with it."""
    w_max = 10.0 if spread == 0.0 else spread / 4.0
    tau = W.uniform_tau(0.05, 1.6, n_tau) if spread == 0.0 else np.linspace(0.0, 4.0, n_tau)
    tgt = W.Target([0.15 * w_max, 0.4 * w_max], [0.04 * w_max, 0.08 * w_max], [0.6, 0.4], w_max)
    wl = W.make(f"sweep-{n_omega}x{n_tau}x{n_walkers}", w_max, n_omega, tau, tgt, 1e-3, 3, n_walkers, n_sweeps, 1e2,
                1.0, n_sweeps, n_sweeps, 5, n_quad=4000)
    if spread > 0.0:
        v = w_max * (tau - tau * tau / 8.0)
        sigma = np.exp(-(v - 0.5 * v.max()))
        wl = dataclasses.replace(wl, sigma=sigma)
    return wl


# bins, times, walkers, precision, walk steps, column spread: which plan of its own it takes
PLANS = [
    (3, 5, 2, 0, 0, 0.0),        # spectra in LDS, fewer bins than a batch of proposals
    (33, 9, 5, 1, 0, 0.0),       # the same in FP32
    (130, 40, 1025, 0, 0, 0.0),  # more than one walker group per compute unit
    (601, 33, 1100, 0, 0, 0.0),  # split, one pair of wavefronts
    (601, 33, 2500, 1, 0, 0.0),  # split, FP32
    (998, 33, 1501, 0, 0, 0.0),  # 16 lanes a walker, spectra in memory
    (998, 33, 4095, 1, 0, 0.0),  # the same in FP32, four pairs
    (1100, 33, 3500, 0, 0, 0.0), # columns fit beside four lanes a walker only
    (1300, 17, 70, 0, 0, 0.0),   # columns larger than LDS
    (130, 40, 8197, 0, 0, 0.0),  # four pairs, whole spectra resident beside them
    (515, 40, 8197, 0, 0, 0.0),  # four pairs, the first bins resident
    (515, 40, 8197, 1, 0, 0.0),  # the same in FP32
    (1023, 20, 8193, 0, 0, 0.0),  # four pairs, no room for columns
    (96, 80, 37, 0, 0, 400.0),   # any number of dimensions
    (96, 80, 37, 1, 0, 400.0),
    (35, 12, 5, 0, 1, 0.0),      # split walk: one step, a remainder of proposals and of walkers
    (35, 12, 1025, 0, 4, 0.0),
    (160, 24, 130, 1, 5, 0.0),   # more steps than are read together
    (3, 5, 2, 0, 9, 0.0),
    (200, 24, 65, 0, 64, 0.0),   # more steps than fit: the walk in its own wavefront
    (700, 24, 4100, 0, 2, 0.0),  # spectra in memory
    (96, 80, 37, 0, 3, 400.0),
]


@pytest.mark.parametrize("n_omega,n_tau,n_walkers,prec,walk,spread", PLANS)
def test_same_bits_for_every_plan(S, n_omega, n_tau, n_walkers, prec, walk, spread):  # noqa: F811
    import torch
    n = 2 if walk > 10 else 7
    wl = _workload(n_omega, n_tau, n_walkers, n, spread)
    side = _workload(40, 11, 19, n)
    sched = S.Schedule(np.geomspace(100.0, 1.0, n), branch_every=n, resync_every=n, walk_len=walk)

    def problem(w, precision):
        gp = S.Problem(w.omega, w.tau, w.Ft, w.sigma, w.m0, w.m1)
        gp.init_walkers(w.n_walkers, 11, precision=precision)
        return gp

    alone, traced, batched = (problem(wl, prec) for _ in range(3))
    alone.run(sched, 0, n)
    flags = torch.zeros((n_walkers, 1, n_omega), dtype=torch.uint8, device="cuda")
    d = torch.zeros((n_walkers, 1, n_omega), dtype=torch.float64, device="cuda")
    traced.set_trace(n - 1, n, d.data_ptr(), flags.data_ptr())
    traced.run(sched, 0, n)
    other = problem(side, 0)
    S.Batch([batched, other]).run([sched, sched], [0, 0], [n, n])
    torch.cuda.synchronize()
    a = alone.read_state()
    assert np.isfinite(a["a"]).all()
    for name, gp in (("traced", traced), ("batch", batched)):
        b = gp.read_state()
        for k in ("a", "F", "rate"):
            np.testing.assert_array_equal(a[k], b[k], err_msg=f"{name}: {k}")
        np.testing.assert_array_equal(alone.read_chi2(), gp.read_chi2(), err_msg=f"{name}: chi2")


@pytest.mark.parametrize("n_omega,n_tau,spread", [(96, 120, 800.0), (96, 120, 1200.0)])
def test_wide_bases_against_oracle(S, n_omega, n_tau, spread):  # noqa: F811
    test_basis_classes_against_oracle(S, n_omega, n_tau, spread)


@pytest.mark.parametrize("n_omega,n_tau,spread", [(60, 7, 0.0), (96, 80, 60.0), (96, 80, 150.0), (96, 80, 250.0),
                                                  (96, 80, 400.0)])
def test_basis_classes_against_oracle(S, n_omega, n_tau, spread):  # noqa: F811
    wl = _workload(n_omega, n_tau, 18, 20, spread)
    _anneal_lockstep(S, wl, 18, 11, 20, dict(branch_every=20, resync_every=10), T=np.geomspace(100.0, 1.0, 20))


def _widening(n_walkers, n_sweeps, prec=0):
    """Weights that turn 500 columns along 512 times into Gaussians which widen
    along tau, the most dimensions of a grid: 98 (FP32: 72) in principal
    directions, 106 (99) as selected.  With prec 1 half the range, scaled so that the
    columns fit a float: 77 in FP32."""
    w_max, tau = 1675.0 / (1 + prec), np.linspace(0.0, 4.0, 512)
    tgt = W.Target([0.15 * w_max, 0.4 * w_max], [0.04 * w_max, 0.08 * w_max], [0.6, 0.4], w_max)
    wl = W.make("widening", w_max, 500, tau, tgt, 1e-3, 3, n_walkers, n_sweeps, 1e2, 1.0, n_sweeps, n_sweeps, 5,
                n_quad=4000)
    slope = np.cumsum((tau / 4.0 + 0.042) ** -1.934)
    slope = w_max * (slope[-1] - slope) / (slope[-1] - slope[0])
    v = np.cumsum(slope) * (tau[1] - tau[0])
    v -= v[-1] - 75.0 if prec else 0.5 * (v[0] + v[-1])
    return dataclasses.replace(wl, sigma=np.exp(-np.clip(v, -340.0, 340.0)))


@pytest.mark.parametrize("n_walkers,prec,walk", [(130, 0, 0), (130, 1, 0), (37, 0, 3), (4500, 1, 0)])
def test_same_bits_for_the_widest_basis(S, monkeypatch, n_walkers, prec, walk):  # noqa: F811
    plain = _workload
    monkeypatch.setattr(sys.modules[__name__], "_workload", lambda o, t, w, n, spread=0.0: (
        _widening(w, n, prec) if spread else plain(o, t, w, n)))
    test_same_bits_for_every_plan(S, 500, 512, n_walkers, prec, walk, 1.0)


# bases of more than 32 dimensions: 16 lanes a walker in every plan
@pytest.mark.parametrize("n_omega,n_tau,n_walkers,prec,walk,spread", [
    (96, 80, 4500, 0, 0, 400.0),   # more walkers than one a wavefront's quarter
    (300, 128, 130, 0, 0, 400.0),  # columns in memory
    (300, 128, 130, 1, 0, 400.0),
    (60, 120, 33, 0, 0, 1100.0),   # as many dimensions as bins, 64 and less
    (96, 120, 33, 0, 0, 1300.0),   # more than 64
    (40, 80, 20, 0, 64, 400.0),    # a walk's steps leave no room for its tables
    (96, 80, 1100, 1, 2, 400.0),
])
def test_same_bits_for_wide_bases(S, n_omega, n_tau, n_walkers, prec, walk, spread):  # noqa: F811
    test_same_bits_for_every_plan(S, n_omega, n_tau, n_walkers, prec, walk, spread)


# jobs, bins, times, walkers, precision, walk steps: launches of many workgroups and their rules
@pytest.mark.parametrize("jobs,n_omega,n_tau,n_walkers,prec,walk", [
    (20, 1300, 17, 1100, 0, 0),  # columns in memory, more workgroups than compute units, a remainder
    (3, 2556, 9, 70, 0, 0),      # room for the bins' table, not the pairs'
    (3, 2556, 9, 70, 1, 0),
    (4, 1100, 17, 300, 0, 0),    # one pair, and wider jobs as far as compute units last
    (4, 1100, 17, 4000, 0, 0),   # more pairs than leave room for the columns
    (24, 40, 12, 700, 0, 2),     # walks of four lanes
    (24, 40, 12, 700, 1, 2),
    (5, 40, 12, 700, 0, 2),      # of eight
    (3, 2000, 9, 40, 0, 1),      # tables beside a walk's records: the bins' only
])
def test_same_bits_in_large_batches(S, jobs, n_omega, n_tau, n_walkers, prec, walk):  # noqa: F811
    n = 2
    wl = _workload(n_omega, n_tau, n_walkers, n)
    sched = S.Schedule(np.geomspace(100.0, 1.0, n), branch_every=n, resync_every=n, walk_len=walk)

    def problem(i):
        gp = S.Problem(wl.omega, wl.tau, wl.Ft, wl.sigma, wl.m0, wl.m1)
        gp.init_walkers(n_walkers, 11 + i, precision=prec)
        return gp

    batched = [problem(i) for i in range(jobs)]
    S.Batch(batched).run([sched] * jobs, [0] * jobs, [1] * jobs)  # ends between resyncs
    for i in sorted({0, 1, jobs // 2, jobs - 1}):
        alone = problem(i)
        alone.run(sched, 0, 1)
        assert alone.state_export() == batched[i].state_export(), f"job {i}"
