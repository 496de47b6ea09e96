"""The two-pass readout stages with several coil chunks per work-group: a last
chunk with fewer coils, a last group with fewer chunks, one and two images,
and lengths whose passes have unequal sizes, against the FP64 oracle with the
FP32 operator's bounds (uncompressed operator: the readout and the
phase-encode DFT alone)."""
import numpy as np
import pytest
import torch

from paper_2601_05418_amd import gpjc, synth
from tests import helpers as H

pytestmark = pytest.mark.gpu


def dev(x):
    return torch.as_tensor(np.ascontiguousarray(x, np.complex64)).cuda()


def check(out, ref):
    torch.cuda.synchronize()
    out = out.cpu().numpy().astype(np.complex128)
    assert H.rel_l2(out, ref) <= H.REL_L2_FP32 and H.max_rel(out, ref) <= 1e-5


# nx, ny, nc, os, batch: enough rows that a work-group takes 2 and more chunks; nc odd, prime, a multiple; os odd, 1
@pytest.mark.parametrize("shape", [(16, 512, 7, 2, 2), (48, 512, 9, 3, 1), (32, 448, 11, 8, 2), (180, 512, 5, 1, 1),
                                   (64, 512, 8, 5, 2), (230, 280, 3, 4, 2)], ids=lambda s: "x".join(map(str, s)))
def test_chunks(gpu_lib, shape):
    nx, ny, nc, os_, batch = shape
    sl = H.rounded_slice(synth._make_rect(3, nx=nx, ny=ny, nc=nc, os_=os_, patch_len=nx, k=1, accel=4, acs=4, cycles=2,
                                          phase_max=2.0))
    g = sl.geom
    plan = gpjc.Plan(g.nx, g.ny, g.nc, g.os, sl.coils, sl.psf, g.mask, batch=batch, compressed=False)
    ops = H.oracle_ops(sl, np.zeros((g.n_groups, 1, nc, nx)))
    rng = np.random.default_rng(5)
    x = H.round64(H.crandn(rng, (batch, ny, nx)))
    y = H.round64(H.crandn(rng, plan.data_shape()))
    f, a = plan.forward(dev(x)), plan.adjoint(dev(y))
    for b in range(batch):
        check(f[b], ops["fwd_full"](x[b]))
        check(a[b], ops["adj_full"](y[b]))
