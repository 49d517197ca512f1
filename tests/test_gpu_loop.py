"""The iteration loop of a solve: graph replays, direct launches and host checks of any length
enqueue exactly the iterations that were asked for."""
from __future__ import annotations

import pytest
import torch

import paper_2511_11359_amd as P
from paper_2511_11359_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("iters", [1, 7, 8, 15, 16, 17, 41])
def test_solve_is_the_same_however_it_is_queued(iters):
    wl = W.random_small(70, 90, 3, seed=3, eta=1e-2)
    prob = P.Problem(wl.x, wl.y, wl.r, wl.c)
    ref = None
    # check_every = 1: two iterations per host check, all launched directly; 9: 18 per check,
    # graph replays and a direct remainder; 64: the default
    for check in (1, 9, 64):
        st, rep, _ = P.solve(prob, P.make_params(eta=wl.eta, max_iter=iters, check_every=check))
        assert rep["iters"] == iters and st.t == iters
        if ref is None:
            ref = st
        assert torch.equal(st.nu, ref.nu) and torch.equal(st.theta, ref.theta)


def test_batch_stops_and_counts_with_the_rest_running():
    wls = [W.random_small(60 + 40 * k, 80, 2, seed=k, eta=1e-2) for k in range(3)]
    mk = lambda: [P.Problem(w.x, w.y, w.r, w.c) for w in wls]  # noqa: E731
    tol = 2e-2
    one = [P.solve(p, P.make_params(eta=1e-2, tol=tol, max_iter=3000))[1] for p in mk()]
    for check in (2, 20):
        states, reps, _ = P.solve_batched(mk(), P.make_params(eta=1e-2, tol=tol, max_iter=3000, check_every=check))
        for s, r, o in zip(states, reps, one):
            assert r["converged"] and r["iters"] == s.t == o["iters"]
            assert r["final_res"] <= tol
