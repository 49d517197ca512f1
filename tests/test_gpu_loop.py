"""The iteration loop of a solve: graph replays, direct launches and host checks of any length
enqueue exactly the iterations that were asked for."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import paper_2511_11359_amd as P
from oracle import lamp as OL
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


@pytest.mark.parametrize("n,m,d,metric", [(1, 1, 1, "sqeuclid"), (63, 65, 2, "sqeuclid"), (64, 129, 3, "l1"), (65, 1031, 7, "sqeuclid"),
                                          (2049, 130, 16, "sqeuclid"), (500, 517, 12, "sqeuclid"), (300, 9, 8, "linf")])
def test_small_sweeps_match_oracle(n, m, d, metric):
    """Small grids run the group-parallel sweeps (64-row blocks, split groups over the waves): ends of
    blocks and groups, fewer groups than waves.  Tolerances as in test_gpu_dims.py."""
    wl = W.random_small(n, m, d, seed=900 + n, eta=1e-2)
    x, y = wl.x.astype(np.float64), wl.y.astype(np.float64)
    s = 1.0 / OL.max_cost(x, y, metric)
    C, prm = OL.ground_cost(x, y, s, metric), OL.Params(eta=wl.eta)
    at, _ = OL.lamp_dense(C, wl.r, wl.c, prm, 3, 1.0, trace=False)
    _, tr_or = OL.lamp_dense(C, wl.r, wl.c, prm, 1, 1.0, state=at)
    dev = lambda v: torch.tensor(v, dtype=torch.float64, device="cuda")  # noqa: E731
    st = P.State(dev(at.nu), dev(at.theta), at.t, at.lam)
    prob = P.Problem(wl.x, wl.y, wl.r, wl.c, cost_scale=s, cost_norm=1.0, metric=metric)
    _, tr = P.step(prob, P.make_params(eta=wl.eta), st, trace=True)
    for col, ref in (("col_a", tr_or.colA[0]), ("col_b", tr_or.colB[0])):
        assert np.all(np.abs(tr[col].cpu().numpy() - ref) <= 4e-6 * ref + 1e-30)
    assert np.max(np.abs(tr["log_za"].cpu().numpy() - tr_or.logZA[0])) <= 2e-6
    assert np.max(np.abs(tr["log_zb"].cpu().numpy() - tr_or.logZB[0])) <= 2e-6


def test_fused_completion_matches_single_steps():
    """A solve completes each iteration in the next one's row pass; steps complete theirs at once.
    From one state, k single iterations resumed by solve(max_iter=1) take the same decisions, and a
    stop keeps the iterate that met the tolerance."""
    wl = W.random_small(130, 210, 2, seed=8, eta=1e-2)
    prob = P.Problem(wl.x, wl.y, wl.r, wl.c)
    full, rep, _ = P.solve(prob, P.make_params(eta=wl.eta, tol=3e-2, max_iter=4000))
    assert rep["converged"] and rep["final_res"] <= 3e-2
    again, rep2, _ = P.solve(prob, P.make_params(eta=wl.eta, max_iter=rep["iters"]))
    assert rep2["iters"] == rep["iters"] == full.t
    assert torch.equal(again.nu, full.nu) and torch.equal(again.theta, full.theta)
    _, rep3, _ = P.solve(prob, P.make_params(eta=wl.eta, tol=3e-2, max_iter=rep["iters"]))
    assert rep3["iters"] == rep["iters"] and not rep3["converged"]   # its iterate is tested one iteration later


@pytest.mark.parametrize("call", ["step", "solve0", "solve1", "solve40", "noalloc", "cert", "batch"])
@pytest.mark.parametrize("fault", ["negative", "nan", "sum"])
def test_bad_marginals_leave_the_state(call, fault):
    """With the cost scale given, step and solve judge the marginals on the device: the call is refused
    and the state is as it was."""
    wl = W.random_small(90, 70, 2, seed=4, eta=1e-2)
    c = wl.c.copy()
    if fault == "sum":
        c *= 1.0 + 1e-8
    else:
        c[33] = -1e-3 if fault == "negative" else float("nan")
    prob = P.Problem(wl.x, wl.y, wl.r, c, cost_scale=0.3, cost_norm=1.0)
    st = P.State(torch.full((70,), 0.01, dtype=torch.float64, device="cuda"),
                 torch.full((70,), 0.02, dtype=torch.float64, device="cuda"), 3, 1.5)
    par = lambda it: P.make_params(eta=1e-2, max_iter=it)  # noqa: E731
    run = {"step": lambda: P.step(prob, par(1), st), "solve0": lambda: P.solve(prob, par(0), st),
           "solve1": lambda: P.solve(prob, par(1), st), "solve40": lambda: P.solve(prob, par(40), st),
           "noalloc": lambda: P.step_noalloc(prob, par(1), st), "cert": lambda: P.certificate(prob, par(1), st),
           "batch": lambda: P.solve_batched([prob, prob], par(9), [st, st.clone()])}[call]
    with pytest.raises(P.LampError) as err:
        run()
    assert err.value.status == -2
    assert ("c[33]" in str(err.value)) == (fault != "sum")
    assert st.t == 3 and torch.all(st.nu == 0.01) and torch.all(st.theta == 0.02)
    good, _, _ = P.solve(P.Problem(wl.x, wl.y, wl.r, wl.c, cost_scale=0.3, cost_norm=1.0), par(3))
    assert good.t == 3 and torch.isfinite(good.nu).all()


def test_solves_on_the_default_stream_from_threads():
    """Calls without a stream take one from the pool, each its own."""
    import threading
    wl = W.random_small(200, 150, 3, seed=6, eta=1e-2)
    ref, _, _ = P.solve(P.Problem(wl.x, wl.y, wl.r, wl.c), P.make_params(eta=1e-2, max_iter=30))
    got = [None] * 6

    def work(k):
        got[k] = P.solve(P.Problem(wl.x, wl.y, wl.r, wl.c), P.make_params(eta=1e-2, max_iter=30))[0]

    ts = [threading.Thread(target=work, args=(k,)) for k in range(6)]
    [t.start() for t in ts]
    [t.join() for t in ts]
    assert all(g is not None and torch.equal(g.nu, ref.nu) for g in got)
