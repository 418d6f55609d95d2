"""The default schedule on both sides of every line of its rule (host code, no
device): lanes per site, workgroup size, streaming access, tile order, the LDS set
aside to limit the workgroups on a CU, and the access of a sweep between two
checks. Any lattice gets a schedule that the kernels take (the call refuses one that
they do not)."""
import random

import pytest

F64, F32 = 0, 1
LIMIT = 54272  # three workgroups of 128 threads on a CU's 160 KB

CACHE = [  # up to 230 MB
    # few sites: four lanes until two fill 512 waves; 8-real eight, four, two
    (F64, 3, 0, (8, 8, 8, 8), (4, 64, 0, 1)), (F64, 3, 0, (10, 10, 10, 10), (4, 64, 0, 1)),
    (F64, 3, 0, (12, 12, 12, 10), (2, 64, 0, 1)), (F64, 3, 2, (8, 8, 8, 8), (8, 64, 0, 1)),
    (F64, 3, 2, (10, 10, 10, 10), (4, 64, 0, 1)), (F64, 3, 2, (16, 14, 14, 14), (2, 64, 0, 1)),
    # streaming between 16 and 48 MB
    (F64, 3, 0, (16, 16, 16, 12), (2, 64, 1, 1)), (F64, 3, 0, (18, 18, 18, 16), (2, 64, 0, 1)),
    (F64, 3, 0, (12, 12, 12, 14), (2, 64, 0, 1)), (F64, 3, 0, (14, 14, 12, 14), (2, 64, 1, 1)),
    # 12-real float links from 1.2e5 sites: one lane
    (F32, 3, 1, (18, 18, 18, 20), (2, 64, 1, 1)), (F32, 3, 1, (18, 18, 20, 20), (1, 256, 1, 1)),
    (F32, 3, 1, (18, 18, 20, 22), (1, 256, 1, 1)), (F32, 3, 1, (22, 22, 22, 26), (1, 256, 0, 1)),
    # 128-thread workgroups beyond 4096 waves
    (F32, 3, 0, (22, 22, 22, 24), (2, 64, 0, 1)), (F32, 3, 0, (22, 22, 22, 26), (2, 128, 0, 1)),
    # SU(2) and SU(4)
    (F32, 2, 0, (16, 16, 16, 16), (2, 64, 0, 1)), (F32, 2, 0, (16, 16, 18, 16), (1, 64, 0, 1)),
    (F64, 2, 0, (16, 16, 18, 16), (2, 64, 1, 1)), (F32, 4, 0, (10, 10, 10, 10), (4, 64, 0, 1)),
    (F32, 4, 0, (12, 12, 12, 12), (2, 64, 0, 1)), (F32, 4, 0, (16, 16, 16, 16), (2, 64, 1, 1)),
    (F32, 4, 0, (20, 20, 20, 20), (2, 64, 0, 1)),
]


@pytest.mark.parametrize("prec,nc,store,dims,want", CACHE)
def test_in_the_cache(prec, nc, store, dims, want):
    from paper_1412_1498_amd import gf
    s = gf.host_schedule(prec, dims, nc, store)
    assert s[:4] == want and s[4] == 0 and s[5] == s[2]


BEYOND = [  # + (limit, streaming between two checks)
    (F32, 3, 0, (28, 28, 30, 30), (2, 128, 0, 1, 0, 0)), (F32, 3, 0, (32, 32, 32, 26), (1, 128, 0, 0, LIMIT, 0)),
    (F32, 3, 0, (40, 40, 36, 36), (1, 128, 0, 0, LIMIT, 0)), (F32, 3, 0, (40, 40, 36, 38), (1, 128, 0, 0, LIMIT, 1)),
    (F32, 3, 0, (36, 40, 40, 38), (1, 128, 0, 0, LIMIT, 0)), (F32, 3, 0, (48, 48, 48, 66), (1, 128, 0, 0, LIMIT, 1)),
    (F32, 3, 0, (48, 48, 48, 70), (1, 128, 1, 0, LIMIT, 1)), (F32, 3, 0, (60, 64, 64, 70), (1, 128, 0, 0, LIMIT, 0)),
    (F32, 3, 0, (60, 64, 64, 72), (1, 128, 1, 0, LIMIT, 1)), (F32, 3, 0, (66, 66, 66, 66), (1, 128, 0, 0, LIMIT, 0)),
    (F32, 3, 1, (72, 72, 72, 72), (1, 128, 0, 0, LIMIT, 1)), (F32, 3, 2, (72, 72, 72, 72), (1, 128, 0, 0, 0, 0)),
    (F64, 3, 0, (32, 32, 32, 30), (2, 128, 0, 0, LIMIT, 0)), (F64, 3, 0, (32, 32, 32, 32), (2, 128, 0, 0, LIMIT, 1)),
    (F64, 3, 0, (34, 32, 32, 32), (2, 128, 0, 0, LIMIT, 0)), (F64, 3, 0, (44, 44, 44, 44), (2, 128, 0, 0, LIMIT, 1)),
    (F64, 3, 0, (44, 44, 44, 46), (2, 128, 1, 1, LIMIT, 1)), (F64, 3, 0, (46, 44, 44, 46), (1, 128, 1, 0, LIMIT, 1)),
    (F64, 3, 1, (60, 60, 60, 60), (2, 128, 0, 0, LIMIT, 1)), (F64, 3, 1, (64, 64, 64, 64), (2, 128, 1, 0, LIMIT, 1)),
    (F64, 3, 1, (66, 66, 66, 66), (2, 128, 0, 0, LIMIT, 0)), (F64, 3, 2, (48, 48, 48, 48), (2, 64, 0, 0, 0, 0)),
    (F64, 2, 0, (48, 48, 48, 48), (2, 128, 0, 0, 0, 0)), (F64, 2, 0, (56, 56, 56, 56), (2, 128, 1, 0, 0, 1)),
    (F64, 4, 0, (32, 32, 32, 32), (2, 128, 0, 0, 0, 0)), (F64, 4, 0, (36, 36, 36, 36), (2, 128, 0, 1, 0, 0)),
    (F64, 4, 0, (40, 40, 40, 40), (2, 128, 1, 1, 0, 1)),
]


@pytest.mark.parametrize("prec,nc,store,dims,want", BEYOND)
def test_beyond_the_cache(prec, nc, store, dims, want):
    from paper_1412_1498_amd import gf
    assert gf.host_schedule(prec, dims, nc, store) == want


def test_ensembles():
    from paper_1412_1498_amd import gf
    small = [(8, 8, 8, 8), (12, 12, 12, 12)]
    assert gf.host_schedule(F32, small)[3] == 0
    many = [(48, 48, 48, 96)] + [(20, 20, 20, 20)] * 50
    assert gf.host_schedule(F32, many) == (1, 128, 1, 0, LIMIT, 1)
    assert gf.host_schedule(F64, many) == (1, 128, 1, 0, LIMIT, 1)
    assert gf.host_schedule(F32, [(24, 24, 24, 48)] * 30) == (1, 128, 0, 0, LIMIT, 0)
    assert gf.host_schedule(F64, [(24, 24, 24, 48)] * 5) == (2, 128, 0, 0, LIMIT, 0)


def test_every_lattice_gets_a_schedule():
    from paper_1412_1498_amd import gf
    rng = random.Random(4)
    for _ in range(3000):
        dims = tuple(2 * rng.randint(1, rng.choice([3, 10, 36])) for _ in range(4))
        nc = rng.choice([2, 3, 3, 3, 4])
        store = rng.choice([0, 1, 2]) if nc == 3 else 0
        s = gf.host_schedule(rng.choice([F64, F32]), dims, nc, store)
        assert s[0] >= (2 if nc == 4 else 1)
    with pytest.raises(gf.GFError):
        gf.host_schedule(F32, (3, 4, 4, 4))
    with pytest.raises(gf.GFError):
        gf.host_schedule(F32, (4, 4, 4, 4), 2, 1)
