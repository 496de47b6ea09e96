"""The calibration's Gram assembly and panel-wise tridiagonal reduction at the
edges of their tiles: panels of 16 steps (or K below that), 16-row blocks,
64-column sums and 64 x 64 updates; patches that are not a multiple of four, of
several tiles, and too long for four coil pairs at a time.  Eigenvalues against
the oracle's Gram matrices, and every kept eigenvector's residual against the
same matrix (which holds without gaps in the spectrum).  Bounds: those of the
calibration tests for eigenvalues and unitarity, and for the residual the
library's own limit, 1e-9 of the largest eigenvalue."""
import numpy as np
import pytest

from oracle import compression as oc
from paper_2601_05418_amd import gpjc, synth
from tests import helpers as H

pytestmark = pytest.mark.gpu


def check(nx, os_, nc, p, k):
    sl = H.rounded_slice(synth._make_rect(2, nx=nx, ny=32, nc=nc, os_=os_, patch_len=p, k=k, accel=2, acs=4, cycles=2,
                                          phase_max=2.0))
    g = sl.geom
    plan = gpjc.Plan.from_slice(sl)
    eig, bank = plan.calibrate(want_eigvals=True, want_bank=True)
    bank = bank.cpu().numpy().reshape(g.n_groups, k, nc * p)
    firsts = oc.first_members(g.patch_group, g.n_groups)
    for gi in {0, g.n_groups - 1}:
        pg = oc.gram(oc.virtual_channels(sl.coils, sl.psf, g.os, p, firsts[gi] * p), None)
        lam = np.linalg.eigvalsh(pg)[::-1]
        assert np.max(np.abs(eig[gi] - lam)) <= 1e-10 * lam[0]
        u = bank[gi].conj().T
        assert np.max(np.abs(u.conj().T @ u - np.eye(k))) <= 1e-11
        assert np.linalg.norm(pg @ u - u * eig[gi, :k], axis=0).max() <= 1e-9 * lam[0]


# coils, patch length, K: n = nc P
@pytest.mark.parametrize("shape", [(1, 2, 1), (1, 2, 2), (3, 4, 1), (4, 4, 5), (17, 1, 16), (16, 2, 16), (33, 1, 17),
                                   (8, 8, 3), (65, 1, 20), (10, 16, 24), (33, 8, 16), (29, 16, 40)],
                         ids=lambda s: "x".join(map(str, s)))
def test_reduction_edges(gpu_lib, shape):
    check(32, 2, *shape)


# nx, os, coils, patch length, K
@pytest.mark.parametrize("shape", [(48, 2, 3, 6, 5), (48, 2, 5, 48, 9), (64, 8, 2, 512, 6)],
                         ids=lambda s: "x".join(map(str, s)))
def test_gram_tiles(gpu_lib, shape):
    check(*shape)
