"""The schedule of an ensemble is that of its run: the large members' sweeps go on
when the small ones have converged. A Coulomb lattice of 48^3 x 96 with 64 small
Landau lattices in float (the ensemble of the benchmark) starts with one lane per
site and the large one's streaming access, 4 % faster to the end than what is
fastest while every member is active. The tuner, which times both states and
stays with the context's schedule unless another is faster beyond its runs'
spread, leaves the fields alone, and the tuned run gives the members' own bits."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def test_large_float_ensemble_starts_as_its_largest_member():
    from paper_1412_1498_amd import gf, synth
    members = [(tuple(d), g) for d, g, *_ in synth.ensemble_members(64, seed=0, amp=0.6)]
    ens = gf.Context(None, prec=gf.F32, ensemble=members)
    assert ens.schedule() == dict(lanes_per_site=1, block_threads=128, nontemporal=1, tile_order=0)


@pytest.mark.parametrize("prec", [0, 1])
def test_tuned_ensemble_gives_the_members_own_bits(prec):
    from paper_1412_1498_amd import gf, synth
    members = [((8, 8, 4, 6), gf.LANDAU), ((10, 6, 8, 14), gf.COULOMB), ((4, 4, 4, 4), gf.LANDAU)]
    ens = gf.Context(None, prec=prec, ensemble=members)
    Us, Vs = [], []
    for i, (d, g) in enumerate(members):
        c = gf.Context(d, gauge=g, prec=prec)
        U = c.pack(synth.random_gauge_field(d, 0.4, 20 + i, device="cuda").to(c.cdtype))
        Us.append(U.clone())
        c.sweeps(U, 1.7, 6)
        Vs.append(U)
    before = [u.clone() for u in Us]
    s = ens.autotune(Us, 1.7)
    assert s["tile_order"] == 0 and all(torch.equal(u, v) for u, v in zip(Us, before))
    ens.batch_fix(Us, 1.7, 0.0, 6)
    assert all(torch.equal(u, v) for u, v in zip(Us, Vs))
