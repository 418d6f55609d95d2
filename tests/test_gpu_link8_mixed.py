"""8-real links of the kind without off-diagonal part in row 0 (unit links and
diagonal ones among them) are coded and decoded behind a branch of the whole
wave. A link's bits must not depend on what the other links of its wave are:
fields with one, some and half of such links between ordinary ones, ragged
last block included, give link by link the bits of the two pure fields."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def special(shape, seed):
    """diag(a) with a U(2) block of determinant conj(a); every third the unit matrix."""
    g = torch.Generator().manual_seed(seed)
    z = torch.randn(*shape, 2, 2, generator=g, dtype=torch.float64)
    ph = torch.rand(*shape, generator=g, dtype=torch.float64) * 6 - 3
    z = torch.view_as_complex(z)
    z = z / z.abs().square().sum(-1, keepdim=True).sqrt()
    a = torch.polar(torch.ones_like(ph), ph)
    D = torch.zeros(*shape, 3, 3, dtype=torch.complex128)
    D[..., 0, 0] = a
    D[..., 1, 1], D[..., 1, 2] = z[..., 0], z[..., 1]
    D[..., 2, 1], D[..., 2, 2] = -(a * z[..., 1]).conj(), (a * z[..., 0]).conj()
    D.view(-1, 3, 3)[::3] = torch.eye(3, dtype=torch.complex128)
    return D


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (6, 4, 2, 6), (8, 4, 6, 4)])
@pytest.mark.parametrize("every", [0, 97, 2])
def test_bits_are_the_links_own(prec, dims, every):
    from paper_1412_1498_amd import gf, synth
    ctx = gf.Context(dims, prec=prec, params=gf.default_params(prec, storage=gf.STORE_8))
    R = synth.random_gauge_field(dims, 0.5, 4, device="cuda").to(ctx.cdtype)
    D = special(R.shape[:-2], 5).to(device="cuda", dtype=ctx.cdtype)
    n = R.numel() // 9
    pick = torch.zeros(n, dtype=torch.bool, device="cuda")
    if every: pick[1::every] = True
    else: pick[n // 2] = True
    pick = pick.view(R.shape[:-2])[..., None, None]
    through = [ctx.unpack(ctx.pack(f)) for f in (torch.where(pick, D, R), D, R)]
    assert torch.isfinite(torch.view_as_real(through[1])).all()
    assert torch.equal(through[0], torch.where(pick, through[1], through[2]))
