"""The packers' tiles at the sizes where they can go wrong: fewer half indices
than one tile, a last tile that is partly or wholly past the lattice's end,
whole tiles only; every precision, storage form, colour number, and the
algebra fields. Packing goes into a buffer of NaNs and must leave every value
in its documented place and zeros in the padding; unpacking returns the
canonical field. Copies, so equality is exact."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

# V / 2 = 8, 40 (one tile, part of it), 96 (32 past a block), 64, 128 (whole), 1400 (odd remainder)
SIZES = [(2, 2, 2, 2), (10, 2, 2, 2), (6, 4, 4, 2), (4, 4, 4, 2), (4, 4, 4, 4), (10, 14, 2, 10)]


@pytest.fixture(scope="module")
def gf():
    from paper_1412_1498_amd import gf as mod
    return mod


def places(dims):
    """(parity, half index) of every canonical site [t][z][y][x], flattened."""
    nx, ny, nz, nt = dims
    t, z, y, x = np.meshgrid(*[np.arange(n) for n in (nt, nz, ny, nx)], indexing="ij")
    return ((x + y + z + t) % 2).reshape(-1), ((x + nx * (y + ny * (z + nz * t))) // 2).reshape(-1)


def blocked(a, dims, values):
    """[site][values] -> [parity][block][values][64], zero padded."""
    p, h = places(dims)
    nb = -(-(len(p) // 2) // 64)
    out = np.zeros((2, nb, values) + (64,) + a.shape[2:], dtype=a.dtype)
    out[p, h // 64, :, h % 64] = a
    return out


@pytest.mark.parametrize("dims", SIZES)
@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("nc,store", [(3, 0), (3, 1), (2, 0), (4, 0)])
def test_pack_places_and_padding(gf, dims, prec, nc, store):
    rng = np.random.default_rng(1)
    V = int(np.prod(dims))
    ct = np.complex128 if prec == 0 else np.complex64
    a = (rng.standard_normal((V, 4, nc, nc)) + 1j * rng.standard_normal((V, 4, nc, nc))).astype(ct)
    ctx = gf.Context(dims, prec=prec, nc=nc, params=gf.default_params(prec, storage=store))
    d = dims[::-1]
    A = torch.from_numpy(a.reshape(*d, 4, nc, nc)).cuda()
    ne = 6 if store == 1 else nc * nc
    stored = a.reshape(V, 4, nc * nc)[:, :, :ne].reshape(V, 4 * ne)
    want = blocked(np.stack([stored.real, stored.imag], -1), dims, 4 * ne)
    U = torch.full((2, want.shape[1], 4, ne, 64, 2), float("nan"), dtype=ctx.rdtype, device="cuda")
    ctx.pack(A, U)
    assert np.array_equal(U.cpu().numpy().reshape(want.shape), want)
    assert np.array_equal(ctx.pack(A).cpu().numpy().reshape(want.shape), want)
    back = ctx.unpack(U).cpu().numpy().reshape(V, 4, nc, nc)
    if store == 0:
        assert np.array_equal(back, a)
    else:
        assert np.array_equal(back[:, :, :2], a[:, :, :2])


@pytest.mark.parametrize("dims", SIZES)
@pytest.mark.parametrize("prec", [0, 1])
def test_algebra_places_and_padding(gf, dims, prec):
    rng = np.random.default_rng(2)
    V = int(np.prod(dims))
    a = rng.standard_normal((V, 8)).astype(np.float64 if prec == 0 else np.float32)
    ctx = gf.Context(dims, prec=prec)
    s = ctx.pack_alg(torch.from_numpy(a.reshape(*dims[::-1], 8)).cuda())
    want = blocked(a, dims, 8)
    assert np.array_equal(s.cpu().numpy(), want)
    assert np.array_equal(ctx.unpack_alg(s).cpu().numpy().reshape(V, 8), a)
