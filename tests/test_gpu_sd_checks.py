"""Alg. 2's checks between steps take F and theta from the next step's Delta
pass (sums over site rows); the last one is gf_quality itself. Against
gf_quality after the same steps, on lattices whose last workgroup of rows is
ragged, whose rows hold few and many sites, in every storage form.

The site terms are the same doubles summed in another order: at most 8 terms
in a lane, 6 + 2 levels in a workgroup, then the final sum's lanes (up to 8
terms here), 6 levels and 16 waves, so 46 additions of rounding 2^-53 each:
5.2e-15 of the sum of absolute terms, which is below 1 for F and theta itself
for theta (whose terms are squares)."""
import json

import pytest

pytestmark = pytest.mark.gpu

CASES = [(0, 0, (4, 2, 2, 2), 0), (1, 0, (6, 10, 14, 4), 0), (0, 1, (10, 6, 4, 14), 1), (1, 2, (26, 6, 10, 4), 1),
         (0, 2, (8, 12, 10, 6), 0), (1, 1, (70, 4, 2, 6), 0), (0, 0, (36, 6, 10, 8), 1)]


def setup(prec, store, dims, gauge, **kw):
    from paper_1412_1498_amd import gf, synth
    ctx = gf.Context(dims, gauge=gauge, prec=prec, params=gf.default_params(prec, storage=store, **kw))
    return ctx, ctx.pack(synth.random_gauge_field(dims, 0.3, 8, device="cuda").to(ctx.cdtype))


@pytest.mark.parametrize("prec,store,dims,gauge", CASES)
def test_checks_between_steps(prec, store, dims, gauge, tmp_path):
    log = tmp_path / "sd.jsonl"
    a, U = setup(prec, store, dims, gauge, check_every=2, log_path=str(log))
    b, V = setup(prec, store, dims, gauge)
    r = a.sd_fix(U, 0.05, 0.0, 5)
    want = {0: b.quality(V)}
    for n in range(1, 6):
        b.sd_step(V, 0.05)
        want[n] = b.quality(V)
    rows = [json.loads(x) for x in log.read_text().splitlines()]
    assert [x["step"] for x in rows] == [0, 2, 4, 5]
    for x in rows:
        F, theta = want[x["step"]]
        assert abs(x["F"] - F) <= 5.2e-15 and abs(x["theta"] - theta) <= 5.2e-15 * theta
    assert (r["F"], r["theta"]) == want[5]


@pytest.mark.parametrize("prec,store,dims,gauge", CASES[:4])
def test_a_run_ends_with_the_fields_own_check(prec, store, dims, gauge):
    a, U = setup(prec, store, dims, gauge)
    theta0 = a.quality(U)[1]
    r = a.sd_fix(U, 0.05, 0.3 * theta0, 400)
    assert r["converged"] and 0 < r["iters"] < 400
    assert (r["F"], r["theta"]) == a.quality(U)
    again = a.sd_fix(U, 0.05, 0.3 * theta0, 400)  # already there: no step, the same field
    assert again["converged"] and again["iters"] == 0 and again["theta"] == r["theta"]
    assert a.sd_fix(U, 0.05, 0.0, 0)["theta"] == r["theta"]
