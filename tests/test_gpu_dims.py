"""The compiled vector-ALU sweeps of the dimensions between the tuned ones (9 to 15 for the squared
Euclidean cost, 5 to 8 for l1 / l_inf) against the FP64 oracle: row ranges off the 256-row blocks,
column ranges off the 8-column groups, a few points only."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import paper_2511_11359_amd as P
from oracle import lamp as OL
from paper_2511_11359_amd import workloads as W
from tests.gpu_util import rel_dual, to_np

pytestmark = pytest.mark.gpu

CASES = [(261, 139, 9, "sqeuclid"), (3, 517, 10, "sqeuclid"), (513, 8, 11, "sqeuclid"), (300, 1027, 12, "sqeuclid"),
         (1, 15, 13, "sqeuclid"), (700, 131, 14, "sqeuclid"), (257, 263, 15, "sqeuclid"),
         (259, 141, 5, "l1"), (40, 523, 6, "linf"), (261, 7, 7, "l1"), (129, 270, 8, "linf"), (260, 133, 8, "l1")]


@pytest.mark.parametrize("n,m,d,kind", CASES)
def test_step_matches_oracle(n, m, d, kind):
    """One step from the oracle's state at t = 3 (errors of earlier steps do not enter).  A column
    marginal is within 4e-6 of itself (2e-6 of the normalisers, 1.2e-6 a term, the FP32 sums over 8
    terms), so |d theta_j| <= kappa 4e-6 col_j / c^alpha_j, kappa = 1 and tanh' <= 1."""
    wl = W.random_small(n, m, d, seed=700 + d, eta=1e-2)
    x, y = wl.x.astype(np.float64), wl.y.astype(np.float64)
    s = 1.0 / OL.max_cost(x, y, kind)
    C, prm = OL.ground_cost(x, y, s, kind), OL.Params(eta=wl.eta)
    at, _ = OL.lamp_dense(C, wl.r, wl.c, prm, 3, 1.0, trace=False)
    _, tr_or = OL.lamp_dense(C, wl.r, wl.c, prm, 1, 1.0, state=at)
    prob = P.Problem(wl.x, wl.y, wl.r, wl.c, cost_scale=s, cost_norm=1.0, metric=kind)
    dev = lambda v: torch.tensor(v, dtype=torch.float64, device="cuda")  # noqa: E731
    st = P.State(dev(at.nu), dev(at.theta), at.t, at.lam)
    _, tr = P.step(prob, P.make_params(eta=wl.eta), st, trace=True)
    calpha = wl.c + 0.01 / m
    for col, dual, k in (("col_a", "theta_bar", "A"), ("col_b", "theta_hat", "B")):
        ref = tr_or.colA[0] if k == "A" else tr_or.colB[0]
        step = tr_or.theta_bar[0] if k == "A" else tr_or.theta_hat[0]
        assert np.all(np.abs(to_np(tr[col]) - ref) <= 4e-6 * ref + 1e-30)
        assert np.all(np.abs(to_np(tr[dual]) - step) <= 4e-6 * ref / calpha + 1e-12)
    assert np.max(np.abs(to_np(tr["log_za"]) - tr_or.logZA[0])) <= 2e-6
    assert np.max(np.abs(to_np(tr["log_zb"]) - tr_or.logZB[0])) <= 2e-6


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
