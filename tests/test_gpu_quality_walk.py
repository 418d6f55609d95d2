"""F and theta in double by the kernel that walks a lattice's time slices (t links
passed between lanes), against the one that takes tile by tile (gf_quality_noalloc,
which has no other): the same sites in the same sums, so the results are equal to
the bit. All storage forms and both gauges, runs of slices of one length and of
two, a last run that is shorter, the smallest temporal extent, and the smaller
lattices that walk early (18-real, and 12-real in Landau gauge, with rows that
begin inside a 128-byte line)."""
import ctypes

import pytest
import torch

pytestmark = pytest.mark.gpu

LANDAU, COULOMB = 0, 1
RUN, TILE = 6, 128  # slices per run at most, half indices per tile


def runs(dims):
    st = dims[0] * dims[1] * dims[2] // 2
    assert st % TILE == 0
    return -(-dims[3] // RUN) * (st // TILE)


def check(dims, gauge, storage):
    from paper_1412_1498_amd import gf, synth
    ctx = gf.Context(dims, gauge=gauge, prec=gf.F64, params=gf.default_params(gf.F64, storage=storage))
    U = ctx.pack(synth.random_gauge_field(dims, 0.6, 5, device="cuda"))
    ctx.sweeps(U, 1.7, 1)
    out = torch.full((2,), float("nan"), dtype=torch.float64, device="cuda")
    st = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    assert gf.lib.gf_quality_noalloc(ctypes.c_void_p(U.data_ptr()), (ctypes.c_int * 4)(*dims), gauge, gf.F64, storage,
                                     st, ctypes.c_void_p(out.data_ptr())) == gf.OK
    assert tuple(out.cpu().tolist()) == ctx.quality(U)


@pytest.mark.parametrize("storage", [0, 1, 2])
@pytest.mark.parametrize("gauge", [LANDAU, COULOMB])
@pytest.mark.parametrize("dims", [(64, 64, 44, 14), (64, 64, 64, 8), (64, 64, 128, 2), (48, 48, 48, 32)])
def test_walked_slices_are_the_tiles(dims, gauge, storage):
    # 14 slices in runs of 5, 5, 4; 8 in 4, 4; 2 in one; 32 in 6, 6, 6, 6, 6, 2
    assert runs(dims) >= 2048
    check(dims, gauge, storage)


@pytest.mark.parametrize("gauge,storage", [(LANDAU, 0), (COULOMB, 0), (LANDAU, 1)])
@pytest.mark.parametrize("dims", [(40, 40, 32, 38), (36, 32, 32, 56)])
def test_early_walk(dims, gauge, storage):
    assert 1400 <= runs(dims) < 2048 and dims[0] // 2 % 8
    check(dims, gauge, storage)
