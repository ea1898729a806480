"""GPU: what the basis of the kernel's columns leaves out of a residue change."""
import numpy as np
import pytest

import oracle as O
from paper_1609_07936_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def S():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a visible GPU"
    from paper_1609_07936_amd import sail
    sail.lib()
    return sail


def _recurrence(omega, tau, w, Phi, p, s, dp, ds):
    """sum_i w_i Phi_i s_i with the columns generated along the times by the
    two-term recurrence, sixteen at a time, in doubles."""
    dt = (tau[-1] - tau[0]) / (tau.size - 1)
    z = np.exp(-omega * dt)
    total = np.zeros(p.size)
    for c in range(0, tau.size, 16):
        e = np.exp(-omega * (tau[0] + dt * c))
        s0, s1 = e[p] * dp + e[s] * ds, e[p] * (dp * z[p]) + e[s] * (ds * z[s])
        part = np.zeros(p.size)
        for i in range(c, min(c + 16, tau.size)):
            part = part + Phi[:, i] * (w[i] * s0)
            s0, s1 = s1, (z[p] + z[s]) * s1 - (z[p] * z[s]) * s0
        total += part
    return total


# grids whose columns a basis of 8 dimensions holds to between 2e-8 and 1e-7, and larger ones
@pytest.mark.parametrize("n_omega,n_tau,w_max,tau_hi", [(33, 30, 6.36, 1.25), (38, 39, 7.83, 1.02), (49, 92, 7.1, 1.09),
                                                        (128, 128, 20.0, 3.0), (256, 256, 20.0, 3.0)])
def test_residue_changes_as_exact_as_the_recurrence(S, n_omega, n_tau, w_max, tau_hi):
    """Errors of the residue changes against 80 bits, in units of their
    condition scale, on spectra of two bins, which resolve the columns best: no
    larger than what summing over recurrence-generated columns in doubles leaves
    in one of their terms (2 r sum_i w_i Phi_i s_i)."""
    import torch
    n, seed, ld = 4096, 5, np.longdouble
    tau = W.uniform_tau(0.05, tau_hi, n_tau)
    tgt = W.Target([0.2 * w_max, 0.4 * w_max], [0.04 * w_max, 0.08 * w_max], [0.6, 0.4], w_max)
    wl = W.make("basis", w_max, n_omega, tau, tgt, 1e-4, 3, n, 4, 1e2, 1.0, 100, 100, 5, n_quad=2000)
    omega, dw = wl.omega, wl.omega[1] - wl.omega[0]
    A, B = wl.m0 / dw, wl.m1 / dw
    gp = S.Problem(omega, tau, wl.Ft, wl.sigma, wl.m0, wl.m1)
    gp.init_walkers(n, seed)
    rng = np.random.default_rng(1)
    k = int(np.searchsorted(omega, B / A))
    lo, hi = rng.integers(0, k, n), rng.integers(k, n_omega, n)
    x = (B - omega[lo] * A) / (omega[hi] - omega[lo])
    a = np.zeros((n, n_omega))
    a[np.arange(n), hi], a[np.arange(n), lo] = x, A - x
    blob = bytearray(gp.state_export())
    blob[48:48 + a.nbytes] = a.tobytes()
    blob[-1] ^= 0xFF  # another basis: taken by its spectra
    gp.state_import(bytes(blob))
    d = torch.zeros((n, 1, n_omega), dtype=torch.float64, device="cuda")
    f = torch.zeros((n, 1, n_omega), dtype=torch.uint8, device="cuda")
    gp.set_trace(0, 1, d.data_ptr(), f.data_ptr())
    gp.run(S.Schedule(np.full(4, 1e-3)), 0, 1)
    torch.cuda.synchronize()
    got = d.cpu().numpy()[:, 0, 0]  # each walker's first proposal
    X = np.array([O.philox4x32_10((0, 0, l, 0), (seed, 0)) for l in range(n)], dtype=np.uint64)
    p, s = (((X[:, i] * np.uint64(n_omega)) >> np.uint64(32)).astype(int) for i in (0, 1))
    r = 1.0 - 0.1 * (2.0 * (X[:, 2].astype(np.float64) + 0.5) * 2.0 ** -32 - 1.0)
    gap = np.where(p == s, 1.0, omega[p] - omega[s])
    dp = np.where(p == s, 0.0, (1.0 - r) * (B - A * omega[s]) / gap)
    ds = np.where(p == s, 0.0, -(1.0 - r) * (B - A * omega[p]) / gap)
    K = np.exp(-np.outer(omega.astype(ld), tau.astype(ld)))
    c, w = ld(dw) / (2 * np.pi), 1.0 / wl.sigma.astype(ld) ** 2
    wh, Phit, Phi = w * c * c, wl.Ft / c, a @ K
    kp, ks = dp[:, None] * K[p], ds[:, None] * K[s]
    dF = (r - 1.0)[:, None] * Phi + kp + ks
    exact = (wh * dF * (2 * (Phi - Phit) + dF)).sum(axis=1)
    M = (wh * (np.abs(r - 1.0)[:, None] * Phi + np.abs(kp) + np.abs(ks)) * (2 * Phi + 2 * np.abs(Phit) + np.abs(dF))).sum(axis=1)
    err = np.abs((got - exact) / M).astype(float)
    S2 = _recurrence(omega, tau, wh.astype(float), Phi.astype(float), p, s, dp, ds)
    rec = np.abs(2 * r * (S2 - (wh * Phi * (kp + ks)).sum(axis=1)) / M).astype(float)
    rms = [float(np.sqrt(np.mean(v * v))) for v in (err, rec)]
    print(f"{n_omega}x{n_tau}: rms {rms[0]:.1e} (recurrence {rms[1]:.1e}), max {err.max():.1e} ({rec.max():.1e})", flush=True)
    assert rms[0] <= rms[1] and err.max() <= rec.max()
