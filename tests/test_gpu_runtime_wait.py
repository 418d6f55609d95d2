"""The fix drivers' checks waited for by the runtime's own wait (the way of processes
that asked for yielding or blocking waits, and of contexts that time their
half-sweeps) and by watching the checks' records: the same results, sweep for sweep
and bit for bit."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("every", [1, 4, 30])
def test_results_do_not_depend_on_the_wait(prec, every):
    from paper_1412_1498_amd import gf, synth
    dims = (8, 6, 10, 4)
    ctx = [gf.Context(dims, prec=prec, params=gf.default_params(prec, check_every=every, timing=t)) for t in (0, 1)]
    U0 = ctx[0].pack(synth.random_gauge_field(dims, 0.4, 2, device="cuda").to(ctx[0].cdtype))
    for call in (lambda c, u: c.fix(u, 1.7, 1e-5, 2000), lambda c, u: c.fix(u, 1.7, 0.0, 41),
                 lambda c, u: c.fix(u, 1.7, 1e9, 10), lambda c, u: c.sd_fix(u, 0.08, 1e-5, 2000),
                 lambda c, u: c.sd_fix(u, 0.08, 0.0, 7)):
        out = []
        for c in ctx:
            c.sweep_count = 0
            U = U0.clone()
            out.append((call(c, U), U, c.sweep_count))
        assert out[0][0] == out[1][0] and out[0][2] == out[1][2]
        assert torch.equal(out[0][1], out[1][1])
