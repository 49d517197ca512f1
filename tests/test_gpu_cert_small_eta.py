"""The entropic dual values of a certificate as eta goes to 0: from a few units of the cost's rounding down
they are the hard minima's (def:dual_spp) to within eta ln m, at every eta > 0 that a call takes."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import paper_2511_11359_amd as P
from oracle import lamp as OL
from paper_2511_11359_amd import workloads as W

pytestmark = pytest.mark.gpu

ETAS = [1e-9, 1e-15, 1e-17, 1e-18, 1e-20, 1e-30, 1e-300]


def _state(C, wl):
    at, _ = OL.lamp_dense(C, wl.r, wl.c, OL.Params(eta=wl.eta), 12, 1.0, trace=False)
    dev = lambda v: torch.tensor(v, dtype=torch.float64, device="cuda")  # noqa: E731
    return at, P.State(dev(at.nu), dev(at.theta), at.t, at.lam)


def _check(prob, C, at, st, r, c, eta, d):
    # The softmin is 1-Lipschitz in the largest change of C + K v, and lies in [min - eta ln m, min].  An entry
    # is at most 1 and s |x~|^2 at most 9/4, so that d products and a few sums round by (d + 8) 2^-52 of 9/4
    # on each side; the FP32 exponentials move a row's sum by 2e-6 of itself.
    tol = 2e-6 * eta + 9.0 * (d + 8) * 2.0 ** -53
    cert = P.certificate(prob, P.make_params(eta=eta), st)
    for v, key in ((at.theta, "theta"), (at.nu, "nu")):
        t = C + 2.0 * v[None, :]
        mn = t.min(1)
        soft = mn - eta * np.log(np.exp(-(t - mn[:, None]) / eta).sum(1))
        want = float(r @ soft - 2.0 * c @ v)
        assert abs(cert["dual_eta_" + key] - want) <= tol, key
        assert abs(cert["dual_eta_" + key] - cert["dual_" + key]) <= eta * np.log(len(v)) + tol, key


@pytest.mark.parametrize("n,m,d,kind", [(200, 300, 3, "sqeuclid"), (70, 263, 19, "sqeuclid"), (130, 77, 131, "sqeuclid"),
                                        (90, 520, 3, "l1"), (40, 77, 9, "l1"), (90, 33, 11, "linf")])
def test_points(n, m, d, kind):
    wl = W.random_small(n, m, d, seed=160 + d, eta=1e-2)
    x, y = wl.x.astype(np.float64), wl.y.astype(np.float64)
    s = 1.0 / OL.max_cost(x, y, kind)
    C = OL.ground_cost(x, y, s, kind)
    at, st = _state(C, wl)
    prob = P.Problem(wl.x, wl.y, wl.r, wl.c, cost_scale=s, cost_norm=1.0, metric=kind)
    for eta in ETAS:
        _check(prob, C, at, st, wl.r, wl.c, eta, d)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16, torch.float16])
def test_cost_matrix(dtype):
    wl = W.random_small(130, 301, 3, seed=44, eta=1e-2)
    x, y = wl.x.astype(np.float64), wl.y.astype(np.float64)
    mat = torch.tensor(OL.ground_cost(x, y, 1.0, "sqeuclid"), dtype=dtype)
    full = mat.double().numpy()
    s = 1.0 / float(full.max())
    at, st = _state(s * full, wl)
    prob = P.Problem.from_cost(mat.cuda(), wl.r, wl.c, cost_scale=s, cost_norm=1.0)
    for eta in ETAS:
        _check(prob, s * full, at, st, wl.r, wl.c, eta, 1)


@pytest.mark.parametrize("d,kind", [(3, "sqeuclid"), (24, "sqeuclid"), (5, "l1")])
def test_costs_far_above_the_stated_norm(d, kind):
    """What bounds the exponents' parts is the data, whatever cost_norm says: costs of 1e30 at eta = 1e-3 are as
    eta = 1e-33 for costs of 1."""
    wl = W.random_small(90, 76, d, seed=7, eta=1e-2)
    big = 1e15 if kind == "sqeuclid" else 1e30
    prob = P.Problem(wl.x * np.float32(big), wl.y * np.float32(big), wl.r, wl.c, cost_scale=1.0, cost_norm=1.0, metric=kind)
    z = torch.zeros(76, dtype=torch.float64, device="cuda")
    cert = P.certificate(prob, P.make_params(eta=1e-3), P.State(z, z.clone(), 3, 2.5))
    for key in ("theta", "nu"):
        assert cert["dual_eta_" + key] == pytest.approx(cert["dual_" + key], rel=1e-12)
