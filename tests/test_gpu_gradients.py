"""Gradients and transport cost in the dimensions without a packed form: compiled ones (9 to 15, 5 to 8 for
l1 / l_inf) and the run-time form with its chunks of coordinates, against the FP64 oracle."""
from __future__ import annotations

import numpy as np
import pytest

import paper_2511_11359_amd as P
from oracle import lamp as OL
from paper_2511_11359_amd import workloads as W
from tests.gpu_util import rel_inf, to_np

pytestmark = pytest.mark.gpu

CASES = [(261, 139, 9, "sqeuclid"), (7, 517, 15, "sqeuclid"), (1, 9, 17, "sqeuclid"), (300, 8, 33, "sqeuclid"),
         (70, 263, 64, "sqeuclid"), (130, 300, 70, "sqeuclid"), (40, 50, 131, "sqeuclid"), (90, 270, 5, "l1"),
         (33, 141, 8, "linf"), (260, 70, 9, "l1"), (60, 133, 35, "l1"), (65, 131, 37, "linf")]


@pytest.mark.parametrize("n,m,d,kind", CASES)
def test_gradients_and_cost(n, m, d, kind):
    """A weight is within 2e-6 of itself (FP32 exponential of an FP64 argument) and the sums are FP64, so
    a row's mean target is within 4e-6 of the clouds' extent: 1e-5 of the largest gradient."""
    wl = W.random_small(n, m, d, seed=300 + d, eta=1e-2)
    x, y = wl.x.astype(np.float64), wl.y.astype(np.float64)
    s = 1.0 / OL.max_cost(x, y, kind)
    C = OL.ground_cost(x, y, s, kind)
    prob = P.Problem(wl.x, wl.y, wl.r, wl.c, cost_scale=s, cost_norm=1.0, metric=kind)
    params = P.make_params(eta=wl.eta, max_iter=20)
    st, _, _ = P.solve(prob, params)
    nu = to_np(st.nu)
    gx = OL.envelope_grad_x(x, y, wl.r, s, nu, st.inv_eta, 1.0) if kind == "sqeuclid" else \
        OL.envelope_grad_x_metric(x, y, wl.r, s, nu, st.inv_eta, 1.0, kind)
    assert rel_inf(to_np(P.backward(prob, params, st)), gx) <= 1e-5
    gy = OL.envelope_grad_y(x, y, wl.r, s, nu, st.inv_eta, 1.0, kind)
    assert rel_inf(to_np(P.backward_y(prob, params, st)), gy) <= 1e-5
    e = -st.inv_eta * (C + 2.0 * nu[None, :])
    p = np.exp(e - e.max(1, keepdims=True))
    cost = float((wl.r[:, None] * p / p.sum(1, keepdims=True) * C).sum())
    assert float(P.transport_cost(prob, params, st)) == pytest.approx(cost, rel=1e-5)
