"""The certificate's pair passes where the streamed groups of eight columns and the run-time form's
groups of four coordinates end: against the FP64 oracle, tolerances as in test_gpu_lamp.py."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import paper_2511_11359_amd as P
from oracle import lamp as OL
from paper_2511_11359_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,m,d,kind", [(1, 9, 3, "sqeuclid"), (257, 7, 9, "sqeuclid"), (70, 263, 17, "sqeuclid"),
                                        (300, 129, 19, "sqeuclid"), (65, 90, 131, "sqeuclid"), (40, 77, 9, "l1"),
                                        (90, 33, 11, "linf"), (90, 1200, 3, "l1"), (300, 517, 8, "linf")])
def test_certificate_passes(n, m, d, kind):
    wl = W.random_small(n, m, d, seed=60 + d, eta=1e-2)
    x, y = wl.x.astype(np.float64), wl.y.astype(np.float64)
    s = 1.0 / OL.max_cost(x, y, kind)
    C, prm = OL.ground_cost(x, y, s, kind), OL.Params(eta=wl.eta)
    at, _ = OL.lamp_dense(C, wl.r, wl.c, prm, 12, 1.0, trace=False)
    dev = lambda v: torch.tensor(v, dtype=torch.float64, device="cuda")  # noqa: E731
    st = P.State(dev(at.nu), dev(at.theta), at.t, at.lam)
    cert = P.certificate(P.Problem(wl.x, wl.y, wl.r, wl.c, cost_scale=s, cost_norm=1.0, metric=kind),
                         P.make_params(eta=wl.eta), st)
    e = -at.lam * (C + 2.0 * at.nu[None, :])
    p = np.exp(e - e.max(1, keepdims=True))
    p /= p.sum(1, keepdims=True)
    X = wl.r[:, None] * p
    assert cert["cost"] == pytest.approx(float((C * X).sum()), rel=1e-5)
    assert cert["col_res"] == pytest.approx(float(np.abs(X.sum(0) - wl.c).sum()), abs=1e-6)
    assert cert["row_res"] <= 2e-6
    for v, key in ((at.theta, "theta"), (at.nu, "nu")):
        t = C + 2.0 * v[None, :]
        assert cert["dual_" + key] == pytest.approx(float(wl.r @ t.min(1) - 2.0 * wl.c @ v), rel=1e-9, abs=1e-10)
        mn = t.min(1)
        soft = mn - wl.eta * np.log(np.exp(-(t - mn[:, None]) / wl.eta).sum(1))
        # FP32 exponentials of FP64 arguments: 2e-6 relative of a row's sum, times eta
        assert cert["dual_eta_" + key] == pytest.approx(float(wl.r @ soft - 2.0 * wl.c @ v), abs=2e-6 * wl.eta + 1e-10)
    yj = np.minimum(wl.c / X.sum(0), 1.0)
    X2 = X * yj[None, :]
    dr, dc = wl.r - X2.sum(1), wl.c - X2.sum(0)
    want = (C * X2).sum() + (dr @ C @ dc / np.abs(dr).sum() if np.abs(dr).sum() > 0 else 0.0)
    assert cert["rounded_cost"] == pytest.approx(float(want), rel=1e-5)
