"""The set-up of a batch runs each step once for all its problems (d <= 16; larger ones by themselves):
cost maximum, offsets and the first iteration of every problem against its own call."""
from __future__ import annotations

import numpy as np
import pytest

import paper_2511_11359_amd as P
from paper_2511_11359_amd import workloads as W
from tests.gpu_util import to_np

pytestmark = pytest.mark.gpu

SIZES = [(1, 1, 1), (255, 257, 2), (256, 64, 3), (65, 700, 8), (1030, 9, 16), (40, 130, 17), (300, 90, 40)]


@pytest.mark.parametrize("sizes", [SIZES, SIZES[:1], SIZES[1:5], SIZES[5:]])
def test_batch_sets_up_as_each_problem_alone(sizes):
    """The cost scale is a maximum, exact in any order: equal to the last bit.  One iteration (the new
    iterate lies in the other buffer) sums in other splits: a column marginal is within 4e-6 of itself on
    each side, so the duals are within 8e-6 col_j / c^alpha_j."""
    wls = [W.random_small(n, m, d, seed=n + d, eta=1e-2) for n, m, d in sizes]
    mk = lambda: [P.Problem(w.x, w.y, w.r, w.c) for w in wls]  # noqa: E731
    params = P.make_params(eta=1e-2, max_iter=1)
    states, reps, _ = P.solve_batched(mk(), params)
    for w, prob, s, r in zip(wls, mk(), states, reps):
        one, rep, _ = P.solve(prob, params)
        assert r["cost_scale"] == rep["cost_scale"] and r["cost_norm"] == rep["cost_norm"]
        assert s.t == one.t == 1 and r["iters"] == 1
        _, tr = P.step(prob, params, P.State.fresh(len(w.c)), trace=True)
        col = np.maximum(to_np(tr["col_a"]), to_np(tr["col_b"]))
        tol = 8e-6 * col / (w.c + 0.01 / len(w.c)) + 1e-12
        assert np.all(np.abs(to_np(s.theta) - to_np(one.theta)) <= tol)
        assert np.all(np.abs(to_np(s.nu) - to_np(one.nu)) <= tol)


def test_batch_takes_given_scales_and_names_a_bad_marginal():
    wls = [W.random_small(200, 90, d, seed=d, eta=1e-2) for d in (2, 5, 20)]
    given = [P.Problem(w.x, w.y, w.r, w.c, cost_scale=0.25, cost_norm=1.0) for w in wls]
    _, reps, _ = P.solve_batched(given, P.make_params(eta=1e-2, max_iter=2))
    assert all(r["cost_scale"] == 0.25 and r["iters"] == 2 for r in reps)
    bad = wls[1].c.copy()
    bad[3] = -bad[3]
    given[1] = P.Problem(wls[1].x, wls[1].y, wls[1].r, bad, cost_scale=0.25, cost_norm=1.0)
    with pytest.raises(P.LampError, match=r"c\[3\]"):
        P.solve_batched(given, P.make_params(eta=1e-2, max_iter=2))
