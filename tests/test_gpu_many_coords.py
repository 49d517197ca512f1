"""Gradients of a cloud with 2^32 coordinates and more, against the closed form of a single partner point."""
from __future__ import annotations

import pytest
import torch

import paper_2511_11359_amd as P

pytestmark = pytest.mark.gpu

N, D = (1 << 26) + 37, 64   # N D is above 2^32, the number of threads a launch can take


@pytest.mark.parametrize("side", ["x", "y"])
def test_gradient_past_2_32_coordinates(side):
    """One point on the other side, nu = 0, lam = 1/2: X_i1 = r_i, or X_1j the softmax of -C_1j / 2 over j, and
    the gradient is 2 s X (x_k - y_k).  An FP32 exponential, its row's sum and the result's rounding move it by
    less than 1e-6 of itself."""
    torch.cuda.empty_cache()
    need = 200 << 30   # workspace, points and gradient
    if torch.cuda.mem_get_info()[0] < need:
        pytest.skip("needs 215 GiB of free device memory")
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    big = torch.rand(N, D, generator=g, device="cuda")
    one = torch.rand(1, D, generator=g, device="cuda")
    w = torch.full((N,), 1.0 / N, dtype=torch.float64, device="cuda")
    u = torch.ones(1, dtype=torch.float64, device="cuda")
    s = 1.0 / D
    params = P.make_params(eta=1e-2)
    if side == "x":
        prob = P.Problem(big, one, w, u, cost_scale=s, cost_norm=1.0)
        st = P.State(torch.zeros(1, dtype=torch.float64, device="cuda"), torch.zeros(1, dtype=torch.float64, device="cuda"), 1, 0.5)
        grad = P.backward(prob, params, st)
    else:
        prob = P.Problem(one, big, u, w, cost_scale=s, cost_norm=1.0)
        z = torch.zeros(N, dtype=torch.float64, device="cuda")
        st = P.State(z, z.clone(), 1, 0.5)
        grad = P.backward_y(prob, params, st)
        lw = torch.empty(N, dtype=torch.float64, device="cuda")
        for a in range(0, N, 1 << 22):
            lw[a:a + (1 << 22)] = -0.5 * s * (big[a:a + (1 << 22)].double() - one.double()).square().sum(1)
        w = torch.softmax(lw, 0)
    for a in list(range(0, N, 1 << 24)) + [N - 4096]:   # slices over the whole cloud and its end
        b = slice(a, min(N, a + 4096))
        want = 2.0 * s * w[b, None] * (big[b].double() - one.double())
        assert float((grad[b].double() - want).abs().max()) <= 1e-6 * float(want.abs().max())
    assert bool((grad[-1] != 0).any())
    del prob, grad, big
    torch.cuda.empty_cache()
