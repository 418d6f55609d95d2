"""Alg. 1 with long check periods: a field that is fixed already costs its check
and not the launches of a period (0.7 of a period's time when these were enqueued
ahead of the check), and a run that ends after one period costs that period (1.37
of it before). The shortest of several calls each, in turn. And runs of every
length end at the check that a plain loop of sweeps and gf_quality ends at, for
thresholds before, at and after the predicted end."""
import time

import pytest

pytestmark = pytest.mark.gpu


def setup(dims, prec, every, seed=1):
    from paper_1412_1498_amd import gf, synth
    ctx = gf.Context(dims, prec=prec, params=gf.default_params(prec, check_every=every))
    return ctx, ctx.pack(synth.random_gauge_field(dims, 0.4, seed, device="cuda").to(ctx.cdtype))


def test_no_period_is_thrown_away():
    import torch
    ctx, U0 = setup((8, 8, 8, 8), 1, 150)
    V = U0.clone()
    ctx.sweeps(V, 1.7, 150)
    eps = 1.5 * ctx.quality(V)[1]
    times = {}
    for _ in range(12):
        for name, e, n, iters in (("fixed", 1e9, 10 ** 6, 0), ("period", 0.0, 150, 150), ("ends", eps, 10 ** 6, 150)):
            V.copy_(U0)
            torch.cuda.synchronize()
            t = time.perf_counter()
            r = ctx.fix(V, 1.7, e, n)
            times[name] = min(times.get(name, 1.0), time.perf_counter() - t)
            assert r["iters"] == iters
    print(times)
    assert times["fixed"] < 0.25 * times["period"]
    assert times["ends"] < 1.15 * times["period"]


@pytest.mark.parametrize("prec,every", [(0, 1), (0, 3), (1, 6), (0, 40)])
def test_ends_at_the_same_check(prec, every):
    ctx, U0 = setup((6, 4, 8, 4), prec, every, 3)
    # plain loop; reunitarisation phases as in the driver
    V, checks = U0.clone(), []
    ctx.sweep_count = 0
    for n in range(7):
        checks.append(ctx.quality(V))
        ctx.sweeps(V, 1.7, every)
    for n, (F, theta) in enumerate(checks):
        if theta >= min([t for _, t in checks[:n]], default=1e9):
            continue
        for eps, at in ((1.0001 * theta, n), (theta, None)):
            U = U0.clone()
            ctx.sweep_count = 0
            r = ctx.fix(U, 1.7, eps, 6 * every)
            if at is None:
                at = next((m for m in range(n + 1, 7) if checks[m][1] < eps), 6)
            assert r["iters"] == at * every and ctx.sweep_count == at * every
            assert (r["F"], r["theta"]) == checks[at]
