"""GPU: walker state put in from outside (checkpoints) and read back."""
import struct

import numpy as np
import pytest

from paper_1609_07936_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def S():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a visible GPU"
    from paper_1609_07936_amd import sail
    sail.lib()
    return sail


def _workload(n_omega, n_tau, n_walkers, w_max=10.0, tau_hi=1.6):
    tau = W.uniform_tau(0.05, tau_hi, n_tau)
    tgt = W.Target([1.5, 4.0], [0.4, 0.8], [0.6, 0.4], w_max)
    return W.make("state", w_max, n_omega, tau, tgt, 1e-3, 3, n_walkers, 8, 1e2, 1.0, 100, 100, 5, n_quad=2000)


def _problem(S, wl, precision=0, seed=11, sigma=None):
    gp = S.Problem(wl.omega, wl.tau, wl.Ft, wl.sigma if sigma is None else sigma, wl.m0, wl.m1)
    gp.init_walkers(wl.n_walkers, seed, precision=precision)
    return gp


def _sections(blob):
    """Byte offsets of a checkpoint's sections: spectra, coordinates, scales,
    inverse scales, residues, rates, end; and its header's integers."""
    n, n_omega, n_tau, ntau_pad, precision, row = struct.unpack_from("<6i", blob, 8)
    at = [48, 48 + 8 * n * n_omega]
    at.append(at[-1] + (4 if precision else 8) * n * row)
    for _ in range(4):
        at.append(at[-1] + 8 * n)
    return at, (n, n_omega, n_tau, ntau_pad, precision, row)


@pytest.mark.parametrize("how", ["alone", "traced", "batch", "walk"])
@pytest.mark.parametrize("precision", [0, 1])
def test_infinite_residue_keeps_the_sum_rules(S, how, precision):
    """A walker whose residue is infinite sees residue changes of -infinity:
    they are accepted for moves of two bins, which keep both sums, and never
    for p = s, which would scale the spectrum (a third of 3 bins' proposals)."""
    import torch
    wl = _workload(3, 5, 64)
    n = wl.n_walkers
    gp = _problem(S, wl, precision)
    blob = bytearray(gp.state_export())
    at, _ = _sections(blob)
    blob[at[4]:at[5]] = np.full(n, np.inf).tobytes()
    gp.state_import(bytes(blob))
    sched = S.Schedule(np.full(100, 50.0), walk_len=2 if how == "walk" else 0)
    if how == "traced":
        d = torch.zeros((n, 1, 3), dtype=torch.float64, device="cuda")
        f = torch.zeros((n, 1, 3), dtype=torch.uint8, device="cuda")
        gp.set_trace(0, 1, d.data_ptr(), f.data_ptr())
    if how == "batch":
        S.Batch([gp]).run([sched], [0], [1])
    else:
        gp.run(sched, 0, 1)
    torch.cuda.synchronize()
    a = gp.read_state()["a"]
    dw = wl.omega[1] - wl.omega[0]
    # at most three moves of three bins each, a few roundings a term
    np.testing.assert_allclose(a.sum(axis=1) * dw, wl.m0, rtol=64 * 2.0 ** -53)
    assert not np.isfinite(gp.read_chi2()).any()


def _coordinates(blob):
    at, (n, n_omega, n_tau, ntau_pad, precision, row) = _sections(blob)
    return np.frombuffer(blob[at[1]:at[2]], dtype=np.float32 if precision else np.float64).reshape(n, row).astype(np.float64)


def _assert_coordinates(gp, wl, sigma, precision):
    """|phi|^2 = sum_i w_i F_i^2 whatever the basis (to what the basis leaves out
    of it, squared, and the loop precision's rounding), and the residues are the
    spectra's."""
    st = gp.read_state()
    dw = wl.omega[1] - wl.omega[0]
    F = st["a"] @ (np.exp(-np.outer(wl.omega, wl.tau)) * (dw / (2.0 * np.pi)))
    w = 1.0 / sigma ** 2
    phi = _coordinates(gp.state_export())
    np.testing.assert_allclose((phi ** 2).sum(axis=1), (w * F * F).sum(axis=1), rtol=1e-5 if precision else 1e-11)
    np.testing.assert_allclose(gp.read_chi2(), (w * (F - wl.Ft) ** 2).sum(axis=1), rtol=1e-6)


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("other", ["errors", "dimensions", "format 3", "format 4"])
def test_checkpoint_of_another_basis_is_taken_by_its_spectra(S, other, precision):
    """Coordinates in a basis that is not the problem's, or not known to be, are
    not taken as its own: other errors (also such that the basis has another
    number of dimensions), and the formats without a digest."""
    wl = _workload(40, 24, 33, 25.0, 4.0) if other == "dimensions" else _workload(40, 24, 33)
    n, n_tau = wl.n_walkers, wl.tau.size
    sched = S.Schedule(np.full(100, 1e-3))
    a = _problem(S, wl, precision)
    a.run(sched, 0, 3)  # between resyncs
    blob, st = a.state_export(), a.read_state()
    sigma = wl.sigma
    if other == "errors":
        sigma = wl.sigma * (1.0 + 0.5 * np.cos(np.arange(n_tau)))
    elif other == "dimensions":
        v = 25.0 * (wl.tau - wl.tau ** 2 / 8.0)  # columns like Gaussians along the times: more of them count
        sigma = np.exp(0.5 * v.max() - v)
    else:
        at, (_, _, _, ntau_pad, _, _) = _sections(blob)
        phi = blob[at[1]:at[2]]
        if other == "format 3":
            dw = wl.omega[1] - wl.omega[0]
            rows = np.zeros((n, ntau_pad), dtype=np.float32 if precision else np.float64)
            rows[:, :n_tau] = st["F"] / (dw / (2.0 * np.pi))
            phi = rows.tobytes()
        head = bytearray(blob[:48])
        head[7:8] = other[-1:].encode()
        if other == "format 3":
            head[28:32] = struct.pack("<i", 0)
        blob = bytes(head) + blob[48:at[1]] + phi + blob[at[2]:at[6]]
    b = _problem(S, wl, precision, seed=999, sigma=sigma)
    if precision == 0:
        assert (_sections(b.state_export())[1][5] != _sections(a.state_export())[1][5]) == (other == "dimensions")
    b.state_import(blob)
    np.testing.assert_array_equal(b.read_state()["rate"], st["rate"])
    np.testing.assert_allclose(b.read_state()["a"], st["a"], rtol=1e-15)
    _assert_coordinates(b, wl, sigma, precision)
    if other.startswith("format") and precision == 0:
        # the same decisions, for a few sweeps, and so the same spectra
        a.run(sched, 3, 3)
        b.run(sched, 3, 3)
        np.testing.assert_allclose(b.read_state()["a"], a.read_state()["a"], rtol=1e-9)


@pytest.mark.parametrize("precision", [0, 1])
def test_checkpoint_of_the_same_basis_keeps_its_bits(S, precision):
    """Import and export give the same file, also with another padding of the
    times (which no section of it depends on)."""
    wl = _workload(40, 24, 33)
    a = _problem(S, wl, precision)
    a.run(S.Schedule(np.full(100, 1e-3)), 0, 3)
    blob = a.state_export()
    b = S.Problem(wl.omega, wl.tau, wl.Ft, wl.sigma, wl.m0, wl.m1)
    b.set_tau_per_lane(8)
    b.init_walkers(wl.n_walkers, 999, precision=precision)
    assert a.layout() != b.layout()
    b.state_import(blob)
    again = b.state_export()
    assert blob[:20] + blob[24:] == again[:20] + again[24:]  # (bytes 20 to 23 hold the padding)
    b.state_import(blob + b"\0" * 16)  # a buffer larger than the checkpoint
    with pytest.raises(S.SailError):
        b.state_import(blob[:-1])


def test_autotuned_layouts_do_not_vary(S):
    """Speed does not depend on the nominal layout: the autotuners choose the
    default, not what a timing of equal launches happens to favour."""
    for n_omega in (33, 48, 65, 90, 127, 160):
        wl = _workload(n_omega, 40, 64)
        for precision in (0, 1):
            for alone in (False, True):
                gp = S.Problem(wl.omega, wl.tau, wl.Ft, wl.sigma, wl.m0, wl.m1)
                assert gp.autotune_layout(wl.n_walkers, precision, alone=alone) == 16
                gp.init_walkers(wl.n_walkers, 1, precision=precision)
                assert gp.layout() == (4, 16)


# plans of their own: one workgroup's LDS, spectra in memory, four lanes; more dimensions
@pytest.mark.parametrize("n_omega,n_tau,n_walkers,w_max,tau_hi", [(64, 32, 64, 10.0, 1.6), (998, 33, 700, 10.0, 1.6),
                                                                  (130, 40, 8197, 10.0, 1.6), (40, 24, 33, 25.0, 4.0)])
@pytest.mark.parametrize("precision", [0, 1])
def test_carried_coordinates_follow_the_spectra(S, n_omega, n_tau, n_walkers, w_max, tau_hi, precision):
    """Between resyncs the coordinates that the sweep carries are the spectra's,
    as a resync takes them, up to the roundings of the accepted moves; the
    traced sweep carries the same ones bit for bit, and its flags give the
    acceptance rate."""
    import torch
    wl = _workload(n_omega, n_tau, n_walkers, w_max, tau_hi)
    n = 5
    sched = S.Schedule(np.full(100, 50.0))
    a, b = _problem(S, wl, precision), _problem(S, wl, precision)
    a.run(sched, 0, n)
    d = torch.zeros((n_walkers, n, n_omega), dtype=torch.float64, device="cuda")
    f = torch.zeros((n_walkers, n, n_omega), dtype=torch.uint8, device="cuda")
    b.set_trace(0, n, d.data_ptr(), f.data_ptr())
    b.run(sched, 0, n)
    torch.cuda.synchronize()
    blob = a.state_export()
    assert blob == b.state_export()
    accepted = (f.cpu().numpy() & 1).sum(axis=2)
    rate = np.ones(n_walkers)
    for k in range(n):
        rate = (1.0 - 0.1) * rate + 0.1 * (accepted[:, k] / n_omega)
    np.testing.assert_array_equal(a.read_state()["rate"], rate)
    assert accepted.sum() > 0
    other = bytearray(blob)
    other[-1] ^= 0xFF
    b.state_import(bytes(other))  # taken by its spectra
    K = np.exp(-np.outer(wl.omega, wl.tau)) * ((wl.omega[1] - wl.omega[0]) / (2.0 * np.pi)) / wl.sigma
    size = a.read_state()["a"].sum(axis=1).max() * np.sqrt((K * K).sum(axis=1)).max()
    u = 2.0 ** -24 if precision else 2.0 ** -53
    # a move rounds phi and two columns' terms once each, and the spectrum's two values and scale
    bound = (16.0 * accepted.sum(axis=1).max() + n_omega + 64) * u * size
    err = np.abs(_coordinates(blob) - _coordinates(b.state_export())).max()
    print(f"{n_omega}x{n_tau}x{n_walkers}: {err / size:.1e} of the norm, bound {bound / size:.1e}", flush=True)
    assert 0.0 < err <= bound


# (n_omega, n_tau, w_max, tau_hi, weighted, rms of the error over the last of fifty sweeps with values
# per time in FP32, which the coordinates took the place of)
@pytest.mark.parametrize("n_omega,n_tau,w_max,tau_hi,weighted,before", [
    (64, 32, 10.0, 1.6, True, 5.3e-8), (64, 32, 10.0, 1.6, False, 3.1e-8), (512, 128, 20.0, 3.0, True, 3.7e-8),
    (512, 128, 20.0, 3.0, False, 3.0e-8), (301, 77, 12.0, 3.0, True, 4.7e-8), (128, 40, 3.5, 6.3, True, 3.3e-8)])
def test_fp32_residue_changes_late_in_a_segment(S, n_omega, n_tau, w_max, tau_hi, weighted, before):
    """The FP32 loop's residue changes fifty sweeps after a resync, in lockstep
    with the FP64 oracle: within 1e-5 of their condition scale, and no further
    off than sums over the times' own values were."""
    import oracle as O
    import torch
    n, seed, nw = 50, 11, 24
    tau = W.uniform_tau(0.05, tau_hi, n_tau)
    tgt = W.Target([0.15 * w_max, 0.4 * w_max], [0.04 * w_max, 0.08 * w_max], [0.6, 0.4], w_max)
    wl = W.make("late", w_max, n_omega, tau, tgt, 1e-3, 3, nw, 8, 1e2, 1.0, 100, 100, 5, n_quad=2000)
    sigma = wl.sigma if weighted else None
    T = np.geomspace(30.0, 0.01, n)
    gp = S.Problem(wl.omega, wl.tau, wl.Ft, sigma, wl.m0, wl.m1)
    gp.init_walkers(nw, seed, precision=1)
    d = torch.zeros((nw, n, n_omega), dtype=torch.float64, device="cuda")
    f = torch.zeros((nw, n, n_omega), dtype=torch.uint8, device="cuda")
    gp.set_trace(0, n, d.data_ptr(), f.data_ptr())
    gp.run(S.Schedule(T), 0, n)
    torch.cuda.synchronize()
    an = O.Anneal(O.Problem(wl.omega, wl.tau, wl.Ft, sigma, wl.m0, wl.m1), O.Schedule(T), nw, seed)
    out = an.run(0, n, trace=(0, n), replay=f.cpu().numpy(), band=1e-5)
    assert out["hard_mismatch"] == 0, out["first_mismatch"]
    err = np.abs(d.cpu().numpy() - out["dchi2"]) / np.maximum(out["cond"], 1e-300)
    rms = np.sqrt((err ** 2).mean(axis=(0, 2)))
    print(f"{n_omega}x{n_tau}: rms {rms[0]:.1e} to {rms[-1]:.1e}, most {err.max():.1e}", flush=True)
    assert err.max() <= 1e-5
    assert rms.max() <= 1.5 * before and rms[-1] <= before
