"""The cost maximum and the row offsets at d > 16 on problems large enough for the coarse INT8 products,
against plain FP64 torch: operand widths 32, 64, 128, ragged tiles, points at one distance (every tile
a candidate), coordinates of very different size, a coordinate that is not finite."""
from __future__ import annotations

import pytest
import torch

import paper_2511_11359_amd as P

pytestmark = pytest.mark.gpu


def _clouds(kind, n, m, d):
    g = torch.Generator(device="cuda")
    g.manual_seed(d)
    if kind == "onehot":
        eye = torch.eye(d, device="cuda")
        pick = lambda k: eye[torch.randint(0, d, (k,), generator=g, device="cuda")]  # noqa: E731
        return pick(n), pick(m)
    x = torch.randn(n, d, generator=g, device="cuda")
    y = 0.5 + torch.randn(m, d, generator=g, device="cuda")
    if kind == "outlier":
        y[m // 2] *= 300.0
        x[:, 0] *= 1e-6
    return x, y


# each above the 2^31 padded products from which the coarse pass runs
CASES = [("normal", 9001, 8003, 17), ("normal", 6011, 5900, 64), ("normal", 5003, 4100, 100), ("onehot", 8200, 8300, 24),
         ("outlier", 6100, 5700, 40)]


@pytest.mark.parametrize("kind,n,m,d", CASES)
def test_cost_maximum_and_offsets(kind, n, m, d):
    x, y = _clouds(kind, n, m, d)
    r = torch.full((n,), 1.0 / n, dtype=torch.float64, device="cuda")
    c = torch.full((m,), 1.0 / m, dtype=torch.float64, device="cuda")
    mu = 0.5 * (x[0].double() + y[0].double())
    a, b = x.double() - mu, y.double() - mu
    D = torch.addmm(b.square().sum(1)[None, :], a, b.t().contiguous(), alpha=-2.0) + a.square().sum(1)[:, None]
    prob = P.Problem(x, y, r, c)
    s, md = P.cost_scale(prob)
    # FP64 inner products of d terms of at most |x||y|: d 2^-53 of the largest squared norm, and room
    assert md == pytest.approx(float(D.max()), rel=1e-12)
    # the offsets only enter through exactly compensated sums: log Z of the first two couplings
    st = P.State.fresh(m)
    _, tr = P.step(prob, P.make_params(eta=1e-2), st, trace=True)
    lz = torch.logsumexp(-0.5 * s * D, 1)     # lam_1 = tau1 = 1/2, nubar = 0
    assert float((tr["log_zb"] - lz).abs().max()) <= 2e-6


@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_not_finite_is_reported(bad):
    x, y = _clouds("normal", 6011, 5900, 64)
    y[17, 3] = bad
    n, m = x.shape[0], y.shape[0]
    r = torch.full((n,), 1.0 / n, dtype=torch.float64, device="cuda")
    c = torch.full((m,), 1.0 / m, dtype=torch.float64, device="cuda")
    with pytest.raises(P.LampError):
        P.solve(P.Problem(x, y, r, c, cost_scale=1e-3, cost_norm=1.0), P.make_params(eta=1e-2, max_iter=3))
