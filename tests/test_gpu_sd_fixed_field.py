"""Alg. 2 on a large field that is fixed already takes the check and no step:
the call costs well under a run of one step (it took 0.73 of one when the
direction of a step was computed behind the check; the check's two passes over
the links are 0.42 of it). The shortest of several calls each, in turn."""
import time

import pytest

pytestmark = pytest.mark.gpu


def test_no_direction_is_computed_for_a_fixed_field():
    import torch
    from paper_1412_1498_amd import gf, synth
    dims = (32, 32, 32, 32)
    ctx = gf.Context(dims, prec=gf.F32)
    U = ctx.pack(synth.random_gauge_field(dims, 0.4, 1, device="cuda").to(ctx.cdtype))
    fixed, step = [], []
    for _ in range(12):
        for eps, n, out in ((1e9, 10, fixed), (0.0, 1, step)):
            torch.cuda.synchronize()
            t = time.perf_counter()
            r = ctx.sd_fix(U, 0.01, eps, n)
            out.append(time.perf_counter() - t)
            assert r["iters"] == (0 if eps else 1)
    print(min(fixed), min(step))
    assert min(fixed) < 0.58 * min(step)
