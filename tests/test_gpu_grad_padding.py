"""The gradient kernel writes every value of its output: the sites of a lattice
that fills its last block only partly get the oracle's gradient, the padding
zeros, whatever the buffer held; and an algebra field far from zero, whose
series needs many terms, gives the oracle's gradient as well (tolerances of the
gradient tests: 1e-12 of the largest entry in double, 1e-4 in float)."""
import numpy as np
import pytest
import torch

from oracle import diff

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gf():
    from paper_1412_1498_amd import gf as mod
    return mod


@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (10, 2, 2, 2), (6, 4, 4, 2), (4, 6, 2, 8)])
@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("gauge", [0, 1])
@pytest.mark.parametrize("sigma", [0.0, 0.1, 2.0])
def test_gradient_values_and_padding(gf, field_cache, dims, prec, gauge, sigma):
    from paper_1412_1498_amd import synth
    U = field_cache(dims, 0.4, 90)
    ct, rt = (np.complex128, np.float64) if prec == 0 else (np.complex64, np.float32)
    s = (synth.random_algebra_field(dims, 1.0, 91).numpy().reshape(*dims[::-1], 8) * sigma).astype(rt)
    ctx = gf.Context(dims, gauge=gauge, prec=prec)
    Ug = ctx.pack(torch.from_numpy(np.ascontiguousarray(U.astype(ct))).cuda())
    sg = ctx.pack_alg(torch.from_numpy(s).cuda())
    out = torch.full_like(sg, float("nan"))
    ctx.functional_grad(Ug, sg, 1.0, out)
    assert torch.isfinite(out).all()
    assert torch.equal(out, ctx.functional_grad(Ug, sg, 1.0))
    V = int(np.prod(dims))
    assert torch.equal(ctx.pack_alg(ctx.unpack_alg(out)), out) and out.numel() >= 8 * V  # zeros in the padding
    want = diff.gradient(U.astype(ct).astype(np.complex128), s.astype(np.float64), gauge)
    got = ctx.unpack_alg(out).cpu().numpy().astype(np.float64)
    assert np.abs(got - want.reshape(got.shape)).max() <= (1e-12 if prec == 0 else 1e-4) * np.abs(want).max()
