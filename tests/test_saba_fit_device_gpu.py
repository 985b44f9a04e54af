"""The fit's device steps at the edges of its launches: one round, a quad's
remainder, exactly one and just past one pass of a block and of the grid, every
width of a lane's budgets, and step limits below, at and past a queue of launches.

Against a float64 evaluation of the same objective at the returned point (sums of
at most 2 million terms: 1e-9 relative) and, for the step limits, against the same
fit stopped at another limit: the first n steps do not depend on the limit."""
import os
import sys

import numpy as np
import pytest

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
import oracle.saba_fit as F  # noqa: E402
import synthetic as S  # noqa: E402

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def fit(r, phi0, max_iter):
    import paper_2608_20375_amd as G
    T = lambda k: torch.from_numpy(np.ascontiguousarray(r[k])).cuda()
    return G.saba_fit(r["budgets"], T("state"), T("prefix"), T("accepted"), T("latency"),
                      r["tau_min"], phi0, max_iter=max_iter)


@pytest.mark.parametrize("rounds", [1, 3, 127, 128, 129, 32768, 32769])
@pytest.mark.parametrize("count", [1, 4, 15, 16, 17, 32, 33, 64])
def test_sums_at_the_returned_point(rounds, count):
    if rounds > 1000 and count not in (17, 64):
        pytest.skip("two widths are enough for the large logs")
    r = S.gen_replay(rounds, grid=tuple(range(16, 16 + 8 * count, 8)), noise=0.05, seed=count)
    phi0 = (10.0, 20.0, 20.0, 20.0)
    got = fit(r, phi0, 0)
    assert got["iterations"] == 0 and not got["converged"]
    assert got["phi"] == [np.float32(v) for v in phi0]
    res = F.gain_residuals(phi0, r["budgets"], r["state"].astype(np.float64), r["accepted"],
                           r["tau_min"])
    assert got["gain_sse"] == pytest.approx(float(res @ res), rel=1e-9, abs=1e-20)
    if rounds >= 3 and count >= 4:
        # 12 points on three unknowns at the least: the normal equations' condition
        # squared costs about half of fp64's digits
        c, sse = F.fit_cost(r["budgets"], r["prefix"], r["latency"])
        np.testing.assert_allclose(got["c"], c, rtol=1e-6)
        assert got["cost_sse"] == pytest.approx(sse, rel=1e-6)


def test_step_limits():
    r = S.gen_replay(3046, noise=0.05, seed=1)
    phi0 = (10.0, 20.0, 20.0, 20.0)
    full = fit(r, phi0, 500)
    n = full["iterations"]
    assert full["converged"] and 34 < n < 500
    assert fit(r, phi0, n) == full
    last = None
    for k in (1, 2, 29, 30, 31, 33, n - 1):     # around a queue of 32 launches
        a = fit(r, phi0, k)
        assert a["iterations"] == k and not a["converged"]
        assert last is None or a["gain_sse"] <= last
        last = a["gain_sse"]
    assert full["gain_sse"] <= last


@pytest.mark.parametrize("rounds,count,prefix", [(1, 4, 777), (200, 31, 1003), (129, 16, 4095),
                                                 (50, 64, 333), (3046, 8, 1001),
                                                 (200, 1, None), (3046, 1, None)])
def test_cost_of_a_log_that_does_not_determine_it(rounds, count, prefix):
    """Logs of one prefix length, or of one budget: a column of [1, B, B prefix] is a
    multiple of another, and of these sums (whole numbers, exact in fp64) elimination
    leaves a zero pivot, so the cost is reported as zero and not as noise."""
    r = S.gen_replay(rounds, grid=tuple(range(33, 33 + 8 * count, 8)), noise=0.05, seed=count)
    if prefix:
        r["prefix"][:] = prefix
    got = fit(r, (10.0, 20.0, 20.0, 20.0), 5)
    assert got["c"] == [0.0, 0.0, 0.0] and got["cost_sse"] == 0.0
    assert np.isfinite(got["phi"]).all()
