"""The row offsets and the cost maximum of the coarse INT8 passes themselves, on data that they keep and data on
which they are given up (points that repeat, an outlier, a tight half, one-hot features), with a coordinate that is
not finite, and in a batch."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import paper_2511_11359_amd as P
from paper_2511_11359_amd import workloads as W
from tests.gpu_util import to_np

pytestmark = pytest.mark.gpu


def _clouds(kind, n, m, d):
    g = torch.Generator(device="cuda")
    g.manual_seed(d)
    pick = lambda rows, k: rows[torch.randint(0, len(rows), (k,), generator=g, device="cuda")]  # noqa: E731
    if kind == "onehot":
        eye = torch.eye(d, device="cuda")
        return pick(eye, n), pick(eye, m)
    x = torch.randn(n, d, generator=g, device="cuda")
    y = 0.5 + torch.randn(m, d, generator=g, device="cuda")
    if kind == "repeat":
        x, y = pick(x[:64], n), pick(y[:64], m)
    elif kind == "outlier":
        y[m // 2] *= 200.0
    elif kind == "tight":
        x[n // 2:] *= 1e-5
        y[m // 2:] *= 1e-5
    return x.contiguous(), y.contiguous()


def _uniform(k):
    return torch.full((k,), 1.0 / k, dtype=torch.float64, device="cuda")


# (n, m, d) above 2^31 padded products; the first k rows alone are below, so that the FP64 pass finds their extremes.
SIZES = [(16350, 8150, 24, 8150), (8150, 8150, 64, 4096), (8150, 8191, 100, 1024)]


# Eight 16-column tiles share their FP32 sums in a row sweep, and every split of these is a multiple of eight
# (128 coordinates leave no such pair of sizes).
@pytest.mark.parametrize("n,m,d,k", SIZES[:2])
@pytest.mark.parametrize("kind", ["normal", "outlier", "onehot", "repeat", "tight"])
def test_offsets_are_those_of_the_fp64_pass(kind, n, m, d, k):
    """A row's offset cancels from its normaliser except through the FP32 rounding of every exponent, 2^-25 of it a
    term: the same offsets give the same terms, whose FP64 sums differ by their order (1e-15 and the logarithm's
    last bits), and other ones differ by 1e-9 and more."""
    x, y = _clouds(kind, n, m, d)
    g = torch.Generator(device="cuda")
    g.manual_seed(7)
    nu = 0.05 * torch.randn(m, dtype=torch.float64, generator=g, device="cuda")
    theta = 0.1 * torch.randn(m, dtype=torch.float64, generator=g, device="cuda")
    s = 1.0 / float((x[:512, None] - y[None, :512]).double().square().sum(2).max())
    params = P.make_params(eta=1e-2)
    traces = []
    for rows in (n, k):
        prob = P.Problem(x[:rows], y, _uniform(rows), _uniform(m), cost_scale=s, cost_norm=1.0)
        _, tr = P.step(prob, params, P.State(nu.clone(), theta.clone(), 3, 8.0), trace=True)
        traces.append(tr)
    for key in ("log_za", "log_zb"):
        a, b = traces[0][key][:k], traces[1][key]
        assert float(((a - b).abs() / b.abs().clamp(min=1.0)).max()) <= 1e-12, key
    prob = P.Problem(x, y, _uniform(n), _uniform(m), cost_scale=s, cost_norm=1.0)
    _, rep, _ = P.solve(prob, P.make_params(eta=1e-2, max_iter=1))
    assert rep["row_fallbacks"] == 0   # an offset that misses its minimum leaves the window of the sums


@pytest.mark.parametrize("n,m,d,k", SIZES)
@pytest.mark.parametrize("kind", ["normal", "outlier", "onehot", "repeat", "tight"])
def test_cost_maximum_is_that_of_the_parts(kind, n, m, d, k):
    """The maximum is exact in any order: equal, to the last bit, to the largest over parts of the rows that the
    FP64 pass takes (the first point, which sets the centre, leads each part)."""
    x, y = _clouds(kind, n, m, d)
    whole = P.cost_scale(P.Problem(x, y, _uniform(n), _uniform(m)))[1]
    parts = []
    for a in range(1, n, k - 1):
        part = torch.cat([x[:1], x[a:a + k - 1]])
        parts.append(P.cost_scale(P.Problem(part, y, _uniform(len(part)), _uniform(m)))[1])
    assert whole == max(parts)


def test_maximum_with_a_coordinate_that_is_not_finite():
    x, y = _clouds("normal", 6011, 5900, 64)
    want = P.cost_scale(P.Problem(x, torch.cat([y[:17], y[18:]]), _uniform(6011), _uniform(5899)))[1]
    y[17, 3] = float("nan")    # no pair of such a point counts
    assert P.cost_scale(P.Problem(x, y, _uniform(6011), _uniform(5900)))[1] == want
    y[17, 3] = float("inf")
    assert P.cost_scale(P.Problem(x, y, _uniform(6011), _uniform(5900)))[1] == float("inf")


@pytest.mark.parametrize("kind", ["normal", "onehot"])
def test_batch_with_problems_of_the_coarse_passes(kind):
    """Such a problem waits for its maximum by itself in the set-up of a batch.  The scale is equal to the last
    bit, the duals as in test_gpu_batch_setup.py."""
    wl = W.random_small(300, 200, 3, seed=5, eta=1e-2)
    clouds = [(wl.x, wl.y), _clouds(kind, 6011, 5900, 64), (wl.y, wl.x), _clouds(kind, 12000, 9000, 20)]
    mk = lambda: [P.Problem(x, y, _uniform(len(x)), _uniform(len(y))) for x, y in clouds]  # noqa: E731
    params = P.make_params(eta=1e-2, max_iter=1)
    states, reps, _ = P.solve_batched(mk(), params)
    for prob, s, r in zip(mk(), states, reps):
        one, rep, _ = P.solve(prob, params)
        assert r["cost_scale"] == rep["cost_scale"] and r["cost_norm"] == rep["cost_norm"]
        assert s.t == one.t == 1 and r["iters"] == 1
        _, tr = P.step(prob, params, P.State.fresh(prob.m), trace=True)
        col = np.maximum(to_np(tr["col_a"]), to_np(tr["col_b"]))
        tol = 8e-6 * col / (1.0 / prob.m + 0.01 / prob.m) + 1e-12
        assert np.all(np.abs(to_np(s.theta) - to_np(one.theta)) <= tol)
        assert np.all(np.abs(to_np(s.nu) - to_np(one.nu)) <= tol)


@pytest.mark.parametrize("n", [191, 192])
def test_maximum_on_both_sides_of_the_fewest_rows(n):
    m, d = 180001, 64
    x, y = _clouds("normal", n, m, d)
    whole = P.cost_scale(P.Problem(x, y, _uniform(n), _uniform(m)))[1]
    parts = [torch.cat([x[:1], x[a:a + 64]]) for a in range(1, n, 64)]
    assert whole == max(P.cost_scale(P.Problem(q, y, _uniform(len(q)), _uniform(m)))[1] for q in parts)
