"""Which fault of a call is reported does not depend on where its marginals are judged: on the host, which
has just read the cost maximum or a range scale, or by the first kernel."""
from __future__ import annotations

import pytest

import paper_2511_11359_amd as P
from paper_2511_11359_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("run", ["solve", "step"])
@pytest.mark.parametrize("given", [True, False])
@pytest.mark.parametrize("bad_mass", [True, False])
def test_bad_marginals_come_before_bad_step_sizes(run, given, bad_mass):
    w = W.random_small(200, 90, 3, seed=1, eta=1e-2)
    c = w.c.copy()
    if bad_mass:
        c[3] = -c[3]
    prob = P.Problem(w.x, w.y, w.r, c, **(dict(cost_scale=0.25, cost_norm=1.0) if given else {}))
    params = P.make_params(eta=0.1, tau1=12.0, max_iter=2)   # tau1 eta = 1.2 > 1
    with pytest.raises(P.LampError, match=r"c\[3\]" if bad_mass else "tau1"):
        P.solve(prob, params) if run == "solve" else P.step(prob, params, P.State.fresh(90))
