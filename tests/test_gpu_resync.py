"""GPU: the resync's matrix tiles and workgroup sizes, and the branching
search's workgroup shapes, at their edges."""
import numpy as np
import pytest

from paper_1609_07936_amd import workloads as W

pytestmark = pytest.mark.gpu


def _problem(S, n_omega, n_tau, n_walkers, seed=3, precision=0):
    tau = np.array([0.4]) if n_tau == 1 else W.uniform_tau(0.05, 1.6, n_tau)
    tgt = W.Target([1.5, 4.0], [0.4, 0.8], [0.6, 0.4], 10.0)
    wl = W.make("rs", 10.0, n_omega, tau, tgt, 1e-2, 3, n_walkers, 4, 1e2, 1.0, 2, 2, 5, n_quad=2000)
    gp = S.Problem(wl.omega, wl.tau, wl.Ft, wl.sigma, wl.m0, wl.m1)
    gp.init_walkers(n_walkers, seed, precision=precision)
    return wl, gp


# bins around multiples of 4 and 16, columns (times and basis) around 16 and 48,
# walkers around 8 and 16 a workgroup; 16 a workgroup above 2048 walkers and up to 512 bins
@pytest.mark.parametrize("n_omega,n_tau,n_walkers", [(3, 1, 2), (4, 5, 8), (17, 16, 9), (64, 33, 2049), (511, 24, 2063),
                                                     (512, 49, 2064), (513, 32, 2050), (2556, 7, 9)])
def test_resync_against_numpy(n_omega, n_tau, n_walkers):
    from paper_1609_07936_amd import sail as S
    wl, gp = _problem(S, n_omega, n_tau, n_walkers)
    gp.run(S.Schedule(np.full(4, 50.0), branch_every=4, resync_every=2), 0, 2)  # ends with a resync
    a, chi2 = gp.read_state()["a"], gp.read_chi2()
    dw, u = wl.omega[1] - wl.omega[0], 2.0 ** -53
    K = (np.exp(-np.outer(wl.omega, wl.tau)) * (dw / (2.0 * np.pi))).astype(np.longdouble)
    F = a.astype(np.longdouble) @ K
    w, r = (1.0 / wl.sigma.astype(np.longdouble) ** 2), F - wl.Ft
    # each F carries (N_omega + 4) roundings of positive terms (and the kernel's two), each term of
    # the sum four more and N_tau in adding up; the weights two
    dF = (n_omega + 8) * u * F
    bound = (w * (2.0 * np.abs(r) * dF + dF * dF + (n_tau + 8) * u * r * r)).sum(axis=1)
    assert np.all(np.abs(chi2 - (w * r * r).sum(axis=1)) <= bound)
    # the renormalisation restores both sums to the rounding of a sum of N_omega terms, twice
    for m, x in ((wl.m0, np.ones(n_omega)), (wl.m1, wl.omega)):
        assert np.all(np.abs(a @ x * dw / m - 1.0) <= 4.0 * (n_omega + 8) * u * 10.0 / min(abs(wl.m1 / wl.m0), 1.0))


@pytest.mark.parametrize("n_walkers", [2, 63, 64, 65, 256, 257, 1024, 1025, 4096, 4097])
def test_branch_search_shapes_same_event(n_walkers):
    """The search spread over many workgroups (alone) and in one workgroup (a
    batch) at the populations where the workgroup's shape changes."""
    from paper_1609_07936_amd import sail as S
    sched = S.Schedule(np.full(4, 5.0), branch_every=2, resync_every=2)
    ev, state = [], []
    for batch in (False, True):
        _, gp = _problem(S, 9, 6, n_walkers)
        gp.set_event_log(True)
        if batch:
            S.Batch([gp]).run([sched], [0], [4])
        else:
            gp.run(sched, 0, 4)
        ev.append(gp.read_events(2, multipliers=True))
        state.append(gp.read_state()["a"])
    for k in ("delta", "pr", "z", "status", "m"):
        np.testing.assert_array_equal(ev[0][k], ev[1][k], err_msg=k)
    np.testing.assert_array_equal(state[0], state[1])
