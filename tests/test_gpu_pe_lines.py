"""The phase-encode stages in their two-pass form: lengths of every kind of
split (square, unequal, with a factor of 23, the shortest and the longest), line
counts that leave a last work-group with fewer lines, one to all phase-encode
lines sampled; forward and adjoint operators against the FP64 oracle with the
FP32 operator's bounds, on a random bank."""
import dataclasses

import numpy as np
import pytest
import torch

from paper_2601_05418_amd import gpjc, synth
from tests import helpers as H

pytestmark = pytest.mark.gpu


# ny, K, sampled lines
@pytest.mark.parametrize("shape", [(16, 1, 1), (32, 3, 32), (48, 5, 7), (80, 3, 11), (112, 2, 3), (180, 5, 61), (230, 3, 1),
                                   (230, 3, 230), (256, 3, 85)], ids=lambda s: "x".join(map(str, s)))
def test_forward_adjoint(gpu_lib, shape):
    ny, k, ms = shape
    sl = H.rounded_slice(synth._make_rect(4, nx=16, ny=ny, nc=2, os_=3, patch_len=16, k=k, accel=2, acs=4, cycles=2,
                                          phase_max=2.0))
    rng = np.random.default_rng(ny + ms)
    mask = np.zeros(ny, bool)
    mask[rng.permutation(ny)[:ms]] = True
    sl = dataclasses.replace(sl, geom=dataclasses.replace(sl.geom, mask=mask))
    bank = H.random_bank(sl.geom, 1)
    plan = gpjc.Plan.from_slice(sl)
    plan.set_compression(torch.as_tensor(bank).cuda())
    ops = H.oracle_ops(sl, bank)
    x = H.round64(H.crandn(rng, (ny, 16)))
    y = H.round64(H.crandn(rng, plan.data_shape()))
    for out, ref in ((plan.forward(torch.as_tensor(x.astype(np.complex64)[None]).cuda()), ops["fwd"](x)),
                     (plan.adjoint(torch.as_tensor(y.astype(np.complex64)).cuda()), ops["adj"](y[0]))):
        out = out.cpu().numpy().astype(np.complex128)[0]
        assert H.rel_l2(out, ref) <= H.REL_L2_FP32 and H.max_rel(out, ref) <= 1e-5
