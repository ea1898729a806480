"""GPU: the read-outs (averaged spectrum, residue histogram) at the edges of
their tiles and walker spans, against numpy on the walkers' own state."""
import numpy as np
import pytest

from paper_1609_07936_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_omega,n_walkers", [(3, 2), (31, 33), (32, 512), (33, 513), (65, 1025), (300, 2049)])
def test_averaged_spectrum_and_histogram(n_omega, n_walkers):
    from paper_1609_07936_amd import sail as S
    tgt = W.Target([1.5, 4.0], [0.4, 0.8], [0.6, 0.4], 10.0)
    wl = W.make("ro", 10.0, n_omega, W.uniform_tau(0.05, 1.6, 12), tgt, 1e-3, 3, n_walkers, 4, 1e2, 1.0, 100, 100, 5,
                n_quad=2000)
    gp = S.Problem(wl.omega, wl.tau, wl.Ft, wl.sigma, wl.m0, wl.m1)
    gp.init_walkers(n_walkers, 7)
    gp.run(S.Schedule(np.full(4, 50.0)), 0, 3)  # between resyncs: scales other than 1
    a, chi2 = gp.read_state()["a"], gp.read_chi2()
    # both sums add non-negative terms: relative error below one rounding per term and side
    np.testing.assert_allclose(gp.read_spectrum(), a.mean(axis=0), rtol=2.0 * (n_walkers + 4) * 2.0 ** -53, atol=0)
    v = np.log10(chi2)
    for n_bins, lo, hi in ((1, np.nan, np.nan), (7, np.nan, np.nan), (300, v.min() + 0.1 * np.ptp(v), v.max()),
                           (4096, np.nan, np.nan), (5, np.nan, np.nan)):
        counts = gp.read_chi2_hist(n_bins, lo, hi)
        np.testing.assert_array_equal(gp.read_chi2_hist_noalloc(n_bins, lo, hi), counts)
        assert counts.sum() == n_walkers
        l, h = v.min() if np.isnan(lo) else lo, v.max() if np.isnan(hi) else hi
        # a residue within 1e-9 of an inner edge may be counted on either side
        edges = l + (h - l) * np.arange(1, n_bins) / n_bins
        below = np.cumsum(counts)[:-1]
        assert np.all(below >= (v[None, :] < edges[:, None] - 1e-9).sum(axis=1))
        assert np.all(below <= (v[None, :] < edges[:, None] + 1e-9).sum(axis=1))


def test_read_outs_by_several_threads():
    """Histograms (of growing sizes, so that the kept buffer is replaced),
    averaged spectra and states read by several threads at once equal those
    read one after another."""
    from concurrent.futures import ThreadPoolExecutor

    from paper_1609_07936_amd import sail as S
    n = 600
    tgt = W.Target([1.5, 4.0], [0.4, 0.8], [0.6, 0.4], 10.0)
    wl = W.make("ro", 10.0, 70, W.uniform_tau(0.05, 1.6, 12), tgt, 1e-3, 3, n, 4, 1e2, 1.0, 100, 100, 5, n_quad=2000)
    gp = S.Problem(wl.omega, wl.tau, wl.Ft, wl.sigma, wl.m0, wl.m1)
    gp.init_walkers(n, 7)
    gp.run(S.Schedule(np.full(4, 50.0)), 0, 3)
    v = np.log10(gp.read_chi2())

    def read(i):
        if i % 3 == 0:
            return gp.read_spectrum()
        if i % 3 == 1:
            return gp.read_chi2_hist(1 + 7 * i, v.min() + 0.01 * i, v.max())
        return gp.read_state()["F"]

    with ThreadPoolExecutor(4) as pool:
        together = list(pool.map(read, range(60)))
    for i, got in enumerate(together):
        np.testing.assert_array_equal(got, read(i), err_msg=str(i))


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("n_omega,n_tau,n_walkers", [(3, 1, 2), (17, 16, 9), (40, 33, 2000), (300, 24, 2064), (700, 200, 1100)])
def test_reconstructions_are_the_spectra_s(n_omega, n_tau, n_walkers, precision):
    """F read one copy with the rates, or in passes of the kept rows, against
    K a in 80 bits."""
    from paper_1609_07936_amd import sail as S
    tau = np.array([0.4]) if n_tau == 1 else W.uniform_tau(0.05, 1.6, n_tau)
    tgt = W.Target([1.5, 4.0], [0.4, 0.8], [0.6, 0.4], 10.0)
    wl = W.make("ro", 10.0, n_omega, tau, tgt, 1e-3, 3, n_walkers, 4, 1e2, 1.0, 100, 100, 5, n_quad=2000)
    gp = S.Problem(wl.omega, wl.tau, wl.Ft, wl.sigma, wl.m0, wl.m1)
    gp.init_walkers(n_walkers, 7, precision=precision)
    gp.run(S.Schedule(np.full(4, 50.0)), 0, 3)
    st = gp.read_state()
    K = np.exp(-np.outer(wl.omega, wl.tau).astype(np.longdouble)) * ((wl.omega[1] - wl.omega[0]) / (2.0 * np.pi))
    # positive terms: a rounding each for the scale, the column, the product and the sum, and the loop precision's
    u = 2.0 ** -53
    np.testing.assert_allclose(st["F"], (st["a"].astype(np.longdouble) @ K).astype(float), atol=0,
                               rtol=(n_omega + 8) * u + (2.0 ** -24 if precision else 0.0))
    blob = gp.state_export()
    np.testing.assert_array_equal(np.frombuffer(blob[-8 - 8 * n_walkers:-8]), st["rate"])
