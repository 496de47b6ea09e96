"""The FP32 operator where its contractions do not run on FP16 pairs: K above
512 (the expanding form's Z^T does not fit its LDS), and patches of one sample
on a volume whose coils lie too far apart for 32-bit offsets over a k-tile (the
compressing form alone, so that the two directions take different forms).
Bounds: those of the FP32 operator against the FP64 oracle."""
import dataclasses

import numpy as np
import pytest
import torch

from oracle import volume as ov
from paper_2601_05418_amd import gpjc, synth
from tests import helpers as H

pytestmark = pytest.mark.gpu


def dev(x):
    return torch.as_tensor(np.ascontiguousarray(x, np.complex64)).cuda()


def check(out, ref):
    torch.cuda.synchronize()
    out = out.cpu().numpy().astype(np.complex128)
    rl, mr = H.rel_l2(out, ref), H.max_rel(out, ref)
    print(f"rel_l2={rl:.3e} max_rel={mr:.3e}", flush=True)
    assert rl <= H.REL_L2_FP32 and mr <= 1e-5


# K just past the limit (33 blocks of 16), and a ragged K with an odd patch length
@pytest.mark.parametrize("shape", [(32, 32, 20, 2, 32, 520), (16, 48, 40, 3, 16, 601), (48, 32, 61, 3, 9, 530)],
                         ids=lambda s: "x".join(map(str, s)))
def test_long_k(gpu_lib, shape):
    nx, ny, nc, os_, p, k = shape
    sl = H.rounded_slice(synth._make_rect(2, nx=nx, ny=ny, nc=nc, os_=os_, patch_len=p, k=k, accel=2, acs=4, cycles=2,
                                          phase_max=2.0))
    g = sl.geom
    bank = H.random_bank(g, seed=1)
    plan = gpjc.Plan.from_slice(sl)
    plan.set_compression(torch.as_tensor(bank).cuda())
    ops = H.oracle_ops(sl, bank)
    rng = np.random.default_rng(2)
    x, y = H.round64(H.crandn(rng, (ny, nx))), H.round64(H.crandn(rng, plan.data_shape()))
    check(plan.forward(dev(x[None]))[0], ops["fwd"](x))
    check(plan.adjoint(dev(y))[0], ops["adj"](y[0]))
    check(plan.normal(dev(x[None]))[0], ops["nrm"](x))


def test_far_coils(gpu_lib):
    v = synth.volume(3, n=64, nz=64, nc=2, os_=16, patch_len=1, k=1, ry=2, rz=2, shift=1, cycles=4)
    v = dataclasses.replace(v, image=H.round64(v.image), coils=H.round64(v.coils), psf=H.round64(v.psf))
    g = v.geom
    bank = H.random_bank(g, seed=3)
    plan = gpjc.Plan.from_volume(v)
    plan.set_compression(torch.as_tensor(bank).cuda())
    args = (v.coils, v.psf, v.mask2, g.os, bank, g.patch_group, g.patch_len)
    rng = np.random.default_rng(4)
    x, y = H.round64(H.crandn(rng, v.image.shape)), H.round64(H.crandn(rng, plan.data_shape()))
    fwd = ov.forward(x, *args)
    check(plan.forward(dev(x[None]))[0], fwd)
    check(plan.adjoint(dev(y))[0], ov.adjoint(y[0], *args))
    check(plan.normal(dev(x[None]))[0], ov.adjoint(fwd, *args))
