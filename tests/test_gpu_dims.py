"""The compiled vector-ALU sweeps of the dimensions between the tuned ones (9 to 15 for the squared
Euclidean cost, 5 to 8 for l1 / l_inf) against the FP64 oracle: row ranges off the 256-row blocks,
column ranges off the 8-column groups, a few points only.  Tolerances as in test_gpu_lamp.py."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import paper_2511_11359_amd as P
from oracle import lamp as OL
from paper_2511_11359_amd import workloads as W
from tests.gpu_util import rel_dual, rel_l1, to_np

pytestmark = pytest.mark.gpu

CASES = [(261, 139, 9, "sqeuclid"), (3, 517, 10, "sqeuclid"), (513, 8, 11, "sqeuclid"), (300, 1027, 12, "sqeuclid"),
         (1, 15, 13, "sqeuclid"), (700, 131, 14, "sqeuclid"), (257, 263, 15, "sqeuclid"),
         (259, 141, 5, "l1"), (40, 523, 6, "linf"), (261, 7, 7, "l1"), (129, 270, 8, "linf"), (260, 133, 8, "l1")]


@pytest.mark.parametrize("n,m,d,kind", CASES)
def test_steps_match_oracle(n, m, d, kind):
    wl = W.random_small(n, m, d, seed=700 + d, eta=1e-2)
    x, y = wl.x.astype(np.float64), wl.y.astype(np.float64)
    s = 1.0 / OL.max_cost(x, y, kind)
    _, tr_or = OL.lamp_dense(OL.ground_cost(x, y, s, kind), wl.r, wl.c, OL.Params(eta=wl.eta), 4, 1.0)
    prob = P.Problem(wl.x, wl.y, wl.r, wl.c, cost_scale=s, cost_norm=1.0, metric=kind)
    st = P.State.fresh(m)
    for k in range(4):
        _, tr = P.step(prob, P.make_params(eta=wl.eta), st, trace=True)
        assert rel_l1(to_np(tr["col_a"]), tr_or.colA[k]) <= 1e-6
        assert rel_l1(to_np(tr["col_b"]), tr_or.colB[k]) <= 1e-6
        assert np.max(np.abs(to_np(tr["log_za"]) - tr_or.logZA[k])) <= 2e-6
        assert np.max(np.abs(to_np(tr["log_zb"]) - tr_or.logZB[k])) <= 2e-6
        assert rel_dual(to_np(st.nu), tr_or.nu[k]) <= 1e-6
        assert rel_dual(to_np(st.theta), tr_or.theta[k]) <= 1e-6


def test_batch_of_untuned_dimensions_matches_single_solves():
    """The batch's items run the same bodies: each problem of d = 5, 9, 12, 15 after a few steps
    equals its own solve (splits differ: FP32 group sums, 1e-6 of the dual scale)."""
    wls = [W.random_small(200 + 37 * d, 150 + 11 * d, d, seed=d, eta=1e-2) for d in (5, 9, 12, 15)]
    params = P.make_params(eta=1e-2, max_iter=6)
    states, reps, _ = P.solve_batched([P.Problem(w.x, w.y, w.r, w.c) for w in wls], params)
    for w, s, r in zip(wls, states, reps):
        one, _, _ = P.solve(P.Problem(w.x, w.y, w.r, w.c), params)
        assert r["iters"] == 6 and torch.isfinite(s.nu).all()
        assert rel_dual(to_np(s.nu), to_np(one.nu)) <= 1e-6
        assert rel_dual(to_np(s.theta), to_np(one.theta)) <= 1e-6
