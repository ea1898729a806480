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


def _workload(n_omega, n_tau, n_walkers):
    tau = W.uniform_tau(0.05, 1.6, n_tau)
    tgt = W.Target([1.5, 4.0], [0.4, 0.8], [0.6, 0.4], 10.0)
    return W.make("state", 10.0, n_omega, tau, tgt, 1e-3, 3, n_walkers, 8, 1e2, 1.0, 100, 100, 5, n_quad=2000)


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
