"""Calibration of many coils with one-sample patches: more coil pairs than one
dimension of a grid holds.  Eigenvalues against the Gram matrix of the oracle,
kept eigenvectors by their residual; bounds of the calibration tests."""
import numpy as np
import pytest

from oracle import compression as oc
from paper_2601_05418_amd import gpjc

pytestmark = pytest.mark.gpu


def test_many_coils(gpu_lib):
    nc, n, k = 800, 16, 4
    rng = np.random.default_rng(0)
    c = (rng.standard_normal((nc, n, n)) + 1j * rng.standard_normal((nc, n, n))).astype(np.complex64)
    c *= np.linspace(0.2, 2.0, nc, dtype=np.float32)[:, None, None]
    psf = np.exp(1j * rng.standard_normal((n, n))).astype(np.complex64)
    plan = gpjc.Plan(n, n, nc, 1, c, psf, np.ones(n, bool), 1, np.zeros(n, int), 1, k)
    eig, bank = plan.calibrate(want_eigvals=True, want_bank=True)
    pg = oc.gram(oc.virtual_channels(c.astype(complex), psf.astype(complex), 1, 1, 0), None)
    lam = np.linalg.eigvalsh(pg)[::-1]
    assert np.max(np.abs(eig[0] - lam)) <= 1e-10 * lam[0]
    u = bank.cpu().numpy().reshape(k, nc).conj().T
    assert np.linalg.norm(pg @ u - u * eig[0, :k], axis=0).max() <= 1e-9 * lam[0]
