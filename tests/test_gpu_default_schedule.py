"""The schedule a context picks by lattice size (lanes per site, workgroup
size, access kind, tile order, occupancy limit) gives the bits of a plain
explicit one, on both sides of the rule's lines: lattices of fewer tiles than
XCDs, with ragged last tiles, within the L2s, just above them, and beyond the
last-level cache; ensembles too. The odd half-sweep takes its tiles from the
other end, so a tile left out or taken twice would show."""
import pytest
import torch

pytestmark = pytest.mark.gpu

FORMS = [(prec, store) for prec in (0, 1) for store in (0, 1, 2)]
SIZES = [(2, 2, 2, 2), (4, 6, 2, 8), (10, 6, 4, 14), (8, 8, 8, 8), (12, 12, 12, 12), (16, 14, 18, 16),
         (22, 18, 26, 30)]


@pytest.fixture(scope="module")
def gf():
    from paper_1412_1498_amd import gf as mod
    return mod


def field(gf, dims, prec, seed):
    from paper_1412_1498_amd import synth
    U = synth.random_gauge_field(dims, 0.4, seed, device="cuda")
    return U.to(torch.complex128 if prec == 0 else torch.complex64)


@pytest.mark.parametrize("prec,store", FORMS)
@pytest.mark.parametrize("dims", SIZES)
def test_default_schedule_gives_the_same_bits(gf, dims, prec, store):
    a = gf.Context(dims, prec=prec, params=gf.default_params(prec, storage=store, reunit_every=2))
    b = gf.Context(dims, prec=prec, params=gf.default_params(prec, storage=store, reunit_every=2, lanes_per_site=1,
                                                             block_threads=64, nontemporal=1, tile_order=0))
    U = a.pack(field(gf, dims, prec, 3))
    V = U.clone()
    a.sweeps(U, 1.7, 3)
    b.sweeps(V, 1.7, 3)
    assert torch.equal(U, V), (dims, a.schedule())


@pytest.mark.parametrize("prec", [0, 1])
def test_large_field_takes_the_occupancy_limit_and_the_same_bits(gf, prec):
    dims = (36, 32, 28, 32) if prec == 1 else (28, 26, 28, 24)  # beyond the last-level cache's line of the rule
    a = gf.Context(dims, prec=prec)
    assert a.field_bytes() > 230e6 and a.schedule()["block_threads"] == 128
    b = gf.Context(dims, prec=prec, params=gf.default_params(prec, lanes_per_site=1, block_threads=64, tile_order=0))
    U = a.pack(field(gf, dims, prec, 4))
    V = U.clone()
    a.sweeps(U, 1.7, 2)
    b.sweeps(V, 1.7, 2)
    assert torch.equal(U, V)


def test_ensemble_default_gives_the_members_own_bits(gf):
    members = [((4, 4, 4, 4), gf.LANDAU), ((10, 6, 4, 14), gf.COULOMB), ((8, 8, 8, 8), gf.LANDAU)]
    ens = gf.Context(None, prec=gf.F32, ensemble=members)
    Us, Vs = [], []
    for i, (d, g) in enumerate(members):
        c = gf.Context(d, gauge=g, prec=gf.F32)
        U = c.pack(field(gf, d, 1, 10 + i))
        Us.append(U.clone())
        c.sweeps(U, 1.7, 4)
        Vs.append(U)
    ens.batch_fix(Us, 1.7, 0.0, 4)
    assert all(torch.equal(u, v) for u, v in zip(Us, Vs))


@pytest.mark.parametrize("nc,dims", [(2, (2, 2, 2, 2)), (2, (10, 6, 4, 14)), (2, (16, 14, 18, 16)), (4, (2, 2, 2, 2)),
                                     (4, (10, 6, 4, 14)), (4, (12, 12, 12, 12)), (4, (16, 14, 18, 16))])
@pytest.mark.parametrize("prec", [0, 1])
def test_sun_default_schedule_gives_the_same_bits(gf, nc, dims, prec):
    from paper_1412_1498_amd import synth
    A = synth.random_sun_field(dims, nc, 0.4, 5).to("cuda", torch.complex128 if prec == 0 else torch.complex64)
    out = []
    for kw in ({}, dict(lanes_per_site=2, block_threads=128, nontemporal=1, tile_order=0),
               dict(lanes_per_site=8, block_threads=64, nontemporal=0, tile_order=1)):
        c = gf.Context(dims, prec=prec, nc=nc, params=gf.default_params(prec, reunit_every=2, **kw))
        U = c.pack(A)
        c.sweeps(U, 1.7, 3)
        out.append(U)
    assert torch.equal(out[0], out[1]) and torch.equal(out[0], out[2])
