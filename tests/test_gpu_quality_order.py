"""F and theta of a single lattice, whose tiles are taken in plain order up to
100 MB and in slab blocks beyond, have the bits of the same lattice inside an
ensemble (always plain order): small lattices with a ragged last tile, and
lattices on both sides of the rule's line."""
import pytest
import torch

pytestmark = pytest.mark.gpu

# (prec, storage, dims); 24x24x24x22 float 18-real is 88 MB, 24x24x24x26 104 MB
SIZES = [(1, 0, (4, 6, 2, 8)), (0, 0, (10, 6, 4, 14)), (1, 0, (24, 24, 24, 22)), (1, 0, (24, 24, 24, 26)),
         (1, 1, (28, 24, 26, 30)), (0, 0, (20, 22, 20, 20)), (0, 2, (26, 24, 24, 22)), (0, 2, (28, 24, 26, 24))]


@pytest.mark.parametrize("prec,store,dims", SIZES)
@pytest.mark.parametrize("gauge", [0, 1])
def test_tile_order_keeps_the_bits(prec, store, dims, gauge):
    from paper_1412_1498_amd import gf, synth
    p = gf.default_params(prec, storage=store)
    one = gf.Context(dims, gauge=gauge, prec=prec, params=p)
    ens = gf.Context(None, prec=prec, params=p, ensemble=[(dims, gauge), ((2, 4, 2, 2), gauge)])
    U = synth.random_gauge_field(dims, 0.4, 5, device="cuda").to(one.cdtype)
    V = synth.random_gauge_field((2, 4, 2, 2), 0.4, 6, device="cuda").to(one.cdtype)
    W = one.pack(U)
    small = gf.Context((2, 4, 2, 2), gauge=gauge, prec=prec, params=p).pack(V)
    F, theta = one.quality(W)
    Fs, thetas = ens.batch_quality([W, small])
    assert (F, theta) == (Fs[0], thetas[0])
