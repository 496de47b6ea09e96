"""The FP32 group contractions on FP16 pairs: every column-tile count and split,
ragged tiles in each dimension (K, Ny, the (coil, sample) index), odd patch
lengths, more blocks of K than one step takes, against the FP64 oracle with
the FP32 operator's bounds; and the scaling of the pairs, which has to make
results independent of the data's magnitude."""
import numpy as np
import pytest
import torch

from paper_2601_05418_amd import gpjc, synth
from tests import helpers as H

pytestmark = pytest.mark.gpu
ELEM = 1e-5


def dev(x):
    return torch.as_tensor(np.ascontiguousarray(x, np.complex64)).cuda()


def host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy().astype(np.complex128)


def check(out, ref):
    rl, mr = H.rel_l2(out, ref), H.max_rel(out, ref)
    print(f"rel_l2={rl:.3e} max_rel={mr:.3e}", flush=True)
    assert rl <= H.REL_L2_FP32 and mr <= ELEM


def rect(nx, ny, nc, os_, p, k):
    return H.rounded_slice(synth._make_rect(2, nx=nx, ny=ny, nc=nc, os_=os_, patch_len=p, k=k, accel=2, acs=4, cycles=2,
                                            phase_max=2.0))


# nx, ny, nc, os, P, K: a single tile of everything; K at and past one 16-row tile, past the 80 rows of a work-group,
# past the 5 blocks of a step of the expanding form (K = 97: 7 blocks, K = 200: 13); odd P with a pair that ends a
# coil; P = 1; 18 and 15 row tiles; os 36, whose readout runs on the Stockham form
SHAPES = [(16, 16, 2, 2, 8, 1), (32, 48, 3, 2, 16, 16), (32, 48, 5, 2, 16, 17), (48, 80, 9, 2, 12, 81),
          (32, 32, 13, 2, 8, 97), (32, 48, 14, 2, 16, 200), (48, 48, 5, 3, 9, 11), (48, 80, 7, 2, 3, 20),
          (16, 32, 6, 2, 1, 4), (64, 280, 3, 2, 32, 30), (80, 230, 4, 2, 5, 12), (16, 16, 2, 36, 8, 3)]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_shapes(gpu_lib, shape):
    sl = rect(*shape)
    g = sl.geom
    a = H.random_bank(g, seed=3)
    plan = gpjc.Plan.from_slice(sl, batch=2)
    plan.set_compression(torch.as_tensor(a).cuda())
    ops = H.oracle_ops(sl, a)
    rng = np.random.default_rng(4)
    x = H.round64(H.crandn(rng, (2, g.ny, g.nx)))
    y = H.round64(H.crandn(rng, plan.data_shape()))
    xf, ya = host(plan.forward(dev(x))), host(plan.adjoint(dev(y)))
    for b in range(2):
        check(xf[b], ops["fwd"](x[b]))
        check(ya[b], ops["adj"](y[b]))


@pytest.mark.parametrize("shape", [(48, 80, 9, 2, 12, 40), (48, 80, 7, 3, 9, 20)], ids=["even", "odd"])
def test_every_tile_count_and_split(gpu_lib, shape):
    sl = rect(*shape)
    a = H.random_bank(sl.geom, seed=5)
    plan = gpjc.Plan.from_slice(sl)
    plan.set_compression(torch.as_tensor(a).cuda())
    x = H.round64(H.crandn(np.random.default_rng(6), (1, sl.geom.ny, sl.geom.nx)))
    ref = H.oracle_ops(sl, a)["nrm"](x[0])
    for v in range(plan.gemm_config()["n_compress"]):
        for ks in (1, 2, 3, 8):
            plan.set_gemm_config(v, v, ks)
            check(host(plan.normal(dev(x)))[0], ref)


def test_magnitudes(gpu_lib):
    """Scaling the data or the bank by a power of two scales the result
    exactly, image rows of very different sizes keep their own accuracy,
    zeros give zeros and an infinity does not vanish."""
    sl = rect(48, 80, 9, 2, 12, 40)
    g = sl.geom
    a = H.random_bank(g, seed=7)
    plan = gpjc.Plan.from_slice(sl)
    plan.set_compression(torch.as_tensor(a).cuda())
    ops = H.oracle_ops(sl, a)
    rng = np.random.default_rng(8)
    x = H.round64(H.crandn(rng, (1, g.ny, g.nx)))
    want = plan.normal(dev(x))
    for e in (-70, -20, 20, 70):
        assert torch.equal(plan.normal(dev(x * 2.0 ** e)), want * 2.0 ** e)
    for e in (-30, 30):
        plan.set_compression(torch.as_tensor(a * 2.0 ** e).cuda())
        assert torch.equal(plan.normal(dev(x)), want * 4.0 ** e)
    plan.set_compression(torch.as_tensor(a).cuda())
    xr = H.round64(x * 10.0 ** rng.uniform(-6, 6, (1, g.ny, 1)))
    check(host(plan.normal(dev(xr)))[0], ops["nrm"](xr[0]))
    assert not plan.normal(torch.zeros_like(want)).any()
    bad = dev(x)
    bad[0, 3, 5] = float("inf")
    assert not torch.isfinite(torch.view_as_real(plan.normal(bad))).all()
