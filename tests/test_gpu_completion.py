"""The completion of an iteration adds the residual's block partials in one shape, wherever it runs: in the
next iteration's row finish or in a launch of its own at the end of a host check."""
from __future__ import annotations

import pytest
import torch

import paper_2511_11359_amd as P
from paper_2511_11359_amd import workloads as W

pytestmark = pytest.mark.gpu


# 64 columns a partial: one round of 64 lanes, one and several rounds of the 256 sums, the ends of their groups
@pytest.mark.parametrize("n,m,d", [(300, 4096, 2), (300, 4097, 2), (200, 9000, 2), (70, 16449, 3), (40, 70001, 3),
                                   (30, 270000, 2),
                                   # a row sweep that is waited for past a stop after some of the checks only
                                   (4000, 9000, 3), (700, 4200, 64)])
def test_residual_and_stop_do_not_depend_on_the_host_checks(n, m, d):
    wl = W.random_small(n, m, d, seed=n, eta=1e-2)
    prob = P.Problem(wl.x, wl.y, wl.r, wl.c, cost_scale=0.1, cost_norm=1.0)
    first = []
    for T in (2, 3, 4, 5, 8):   # the residuals of iterates 1 to 7, each completed in a launch of its own
        first.append(P.solve(prob, P.make_params(eta=1e-2, max_iter=T))[1]["final_res"])
    for res in first:
        got = []
        for check in (1, 2, 3, 7, 64):   # a stop at the end of a check or inside it
            st, rep, _ = P.solve(prob, P.make_params(eta=1e-2, tol=res, max_iter=400, check_every=check))
            got.append((rep["iters"], rep["final_res"], st.nu, st.theta))
        assert got[0][1] <= res
        for g in got[1:]:
            assert g[:2] == got[0][:2]
            assert torch.equal(g[2], got[0][2]) and torch.equal(g[3], got[0][3])
