"""Measured cases: what a program built on this package has it do, through the public entry
points of paper_2511_11359_amd (solve, step, certificate, LampOT, solve_batched).

listed() holds named cases, draw(rng) one more of the same ranges, prepare(case, seed) what the
program has in hand before the call (points, marginals, a problem handle, a dual state), run(state)
one pass, work(case) the bytes and operations the pass cannot do without, and exact(case, seed)
the pass's results in FP64 torch, from the definitions and without the library.
"""
import math
import random

import torch

import paper_2511_11359_amd as P

LOG_LO, LOG_HI = math.log(256), math.log(131072)


# ------------------------------------------------------------------ the cases

def listed():
    return [
        # one iteration at a time on a small problem (a serving loop, a parity check): launches and
        # synchronisations count, hardly any arithmetic
        dict(name="step_256_d2", kind="step", n=256, m=256, d=2, cloud="uniform", metric="sqeuclid",
             precision="fp32", marg="uniform", eta=1e-2, t=50),
        # the 4096 x 4096 Gaussian workload: a solve bound by short kernels
        dict(name="solve_4096_d3", kind="solve", n=4096, m=4096, d=3, cloud="gauss", metric="sqeuclid",
             precision="fp32", marg="dirichlet", eta=1e-3, iters=128),
        # embeddings at the headline size, reference-accuracy form and the fast form
        dict(name="solve_65536_d64", kind="solve", n=65536, m=65536, d=64, cloud="gmm", metric="sqeuclid",
             precision="fp32", marg="uniform", eta=1e-3, iters=6),
        dict(name="solve_65536_d64_bf16", kind="solve", n=65536, m=65536, d=64, cloud="gmm", metric="sqeuclid",
             precision="bf16_mfma", marg="uniform", eta=1e-3, iters=24),
        # the split form on ragged sizes and a dimension between the operand widths
        dict(name="solve_40009x30011_d48_fp16x3", kind="solve", n=40009, m=30011, d=48, cloud="gmm",
             metric="sqeuclid", precision="fp16x3_mfma", marg="dirichlet", eta=1e-3, iters=16),
        # large point clouds in space (colour transfer, shapes)
        dict(name="solve_131072_d3", kind="solve", n=131072, m=131072, d=3, cloud="sphere", metric="sqeuclid",
             precision="fp32", marg="uniform", eta=5e-3, iters=6),
        # a dozen features per point, ragged sizes
        dict(name="solve_20011x9973_d12", kind="solve", n=20011, m=9973, d=12, cloud="gmm", metric="sqeuclid",
             precision="fp32", marg="dirichlet", eta=0.0, iters=16),
        # the l1 ground cost
        dict(name="solve_50021x30011_d3_l1", kind="solve", n=50021, m=30011, d=3, cloud="sphere", metric="l1",
             precision="fp32", marg="uniform", eta=1e-3, iters=8),
        # a cost matrix of the caller's, two bytes per entry, rows at odd addresses
        dict(name="solve_cost_40000x50001_bf16", kind="cost", n=40000, m=50001, dtype="bfloat16", eta=0.0, iters=8),
        # a training step: the transport cost and both gradients
        dict(name="autograd_16384x12001_d3", kind="grad", n=16384, m=12001, d=3, cloud="sphere", metric="sqeuclid",
             marg="dirichlet", eta=5e-3, iters=64),
        # many problems of 512 to 8192 points at once
        dict(name="batch_64", kind="batch", count=64, lo=512, hi=8192, dims="2,3,16", eta=1e-3, iters=48),
        # the certificate of a finished solve
        dict(name="certificate_65536_d3", kind="cert", n=65536, m=65536, d=3, cloud="sphere", metric="sqeuclid",
             precision="fp32", marg="uniform", eta=5e-3, t=200),
    ]


def draw(rng):
    """One more case: kinds by how often a program uses them, sizes over the logarithm of their range."""
    kind = rng.choices(["solve", "step", "cost", "grad", "batch", "cert"], [55, 10, 12, 10, 5, 8])[0]
    size = lambda hi: int(round(math.exp(rng.uniform(LOG_LO, math.log(hi)))))  # noqa: E731
    eta = rng.choice([0.0, 1e-3, 5e-3, 1e-2])
    if kind == "batch":
        return dict(kind="batch", count=rng.randint(4, 64), lo=rng.choice([256, 512]), hi=rng.choice([2048, 4096, 8192]),
                    dims=rng.choice(["2,3,16", "2", "3", "2,3", "5,8", "16"]), eta=eta, iters=rng.choice([16, 32, 48]))
    if kind == "cost":
        n, m = size(50000), size(50000)
        return dict(kind="cost", n=n, m=m, dtype=rng.choice(["float32", "bfloat16", "float16"]), eta=eta,
                    iters=rng.choice([4, 8, 16]))
    metric = rng.choices(["sqeuclid", "l1", "linf"], [80, 12, 8])[0]
    d = rng.choice([2, 3]) if rng.random() < 0.5 else int(round(math.exp(rng.uniform(math.log(2), math.log(128)))))
    if metric != "sqeuclid":
        d = min(d, rng.randint(2, 8))
    n, m = size(131072), size(131072)
    cap = 1.7e10 if d <= 3 else 4.3e9 * min(1.0, 16.0 / d)      # pairs
    if kind in ("grad", "cert") and d > 3:
        cap /= 8
    while n * m > cap or max(n, m) > 64 * min(n, m):
        n, m = size(131072), size(131072)
    marg = rng.choice(["uniform", "dirichlet"])
    cloud = rng.choice(["uniform", "gauss", "sphere"]) if d <= 3 else rng.choice(["uniform", "gauss", "gmm"])
    if cloud == "sphere" and d != 3:
        cloud = "gauss"
    c = dict(kind=kind, n=n, m=m, d=d, cloud=cloud, metric=metric, marg=marg, eta=eta)
    if kind in ("solve", "step"):
        forms = ["fp32"] * 6
        if metric == "sqeuclid":
            forms += ["bf16_mfma", "bf16_mfma", "fp16_mfma", "fp32_mfma"] + (["fp16x3_mfma"] * 2 if d <= 64 else [])
        c["precision"] = rng.choice(forms)
    if kind == "cert":
        c["precision"] = "fp32"
    if kind in ("step", "cert"):
        c["t"] = rng.choice([1, 20, 100, 300])
    if kind in ("solve", "grad"):
        c["iters"] = max(2, min(64, int(1.0e11 / (n * m * max(1.0, d / 4.0)))))
        if kind == "grad":
            c["iters"] = min(c["iters"], 32)
    return c


# ------------------------------------------------------------------ inputs

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _normal(g, *shape):
    return torch.randn(*shape, generator=g, device="cuda", dtype=torch.float32)


def _uniform(g, *shape):
    return torch.rand(*shape, generator=g, device="cuda", dtype=torch.float32)


def _clouds(g, cloud, n, m, d):
    """x, y as the package's workloads draw them."""
    if cloud == "gauss":          # N(0, I) against N(1.5, 0.5^2 I)
        return _normal(g, n, d), 1.5 + 0.5 * _normal(g, m, d)
    if cloud == "gmm":            # one 8-component mixture, independent draws
        means = 2.0 * _normal(g, 8, d)
        pick = lambda k: means[torch.randint(0, 8, (k,), generator=g, device="cuda")] + _normal(g, k, d)  # noqa: E731
        return pick(n), pick(m)
    if cloud == "sphere":         # a noisy unit sphere against the unit cube
        v = _normal(g, n, d)
        return v / v.norm(dim=1, keepdim=True) + 0.01 * _normal(g, n, d), _uniform(g, m, d)
    return _uniform(g, n, d), _uniform(g, m, d)


def _marginal(g, kind, k):
    if kind == "uniform":
        return torch.full((k,), 1.0 / k, dtype=torch.float64, device="cuda")
    e = -torch.log1p(-torch.rand(k, generator=g, device="cuda", dtype=torch.float64))
    e = e / e.sum() + 1e-6        # Dirichlet(1) with full support
    return e / e.sum()


def _cost_matrix(case, g):
    """Euclidean distances between points of the plane, in the storage type."""
    x, y = _uniform(g, case["n"], 2), _uniform(g, case["m"], 2)
    out = torch.empty(case["n"], case["m"], dtype=getattr(torch, case["dtype"]), device="cuda")
    for i in range(0, case["n"], 4096):
        a = x[i:i + 4096]
        out[i:i + 4096] = ((a[:, None, 0] - y[None, :, 0]).square_() + (a[:, None, 1] - y[None, :, 1]).square_()).sqrt_()
    return out


def _lam(eta, t, tau1=0.5):
    lam = 0.0
    for _ in range(t):
        lam = tau1 + lam * (1.0 - tau1 * eta)
    return lam


def _batch_sizes(case):
    """(n, m, d) of a batch's problems, log-uniform; the case alone sets them."""
    rng = random.Random(case["count"] * 1000003 + case["hi"])
    dims = [int(v) for v in case["dims"].split(",")]
    size = lambda: int(round(case["lo"] * (case["hi"] / case["lo"]) ** rng.random()))  # noqa: E731
    return [(size(), size(), rng.choice(dims)) for _ in range(case["count"])]


def _inputs(case, seed):
    """The raw inputs of a case, from the seed alone."""
    g = _gen(seed)
    if case["kind"] == "batch":
        return [(_uniform(g, n, d), _uniform(g, m, d), _marginal(g, "dirichlet", n), _marginal(g, "dirichlet", m))
                for n, m, d in _batch_sizes(case)]
    if case["kind"] == "cost":
        cost = _cost_matrix(case, g)
        return cost, _marginal(g, "dirichlet", case["n"]), _marginal(g, "dirichlet", case["m"])
    x, y = _clouds(g, case["cloud"], case["n"], case["m"], case["d"])
    r, c = _marginal(g, case["marg"], case["n"]), _marginal(g, case["marg"], case["m"])
    if case["kind"] not in ("step", "cert"):
        return x, y, r, c
    # a dual state in the middle of a run: nu near the potentials' range, theta inside its clip radius
    duals = [(torch.rand(case["m"], generator=g, device="cuda", dtype=torch.float64) * 2.0 - 1.0) * a for a in (0.01, 0.05)]
    return x, y, r, c, duals[0], duals[1]


def prepare(case, seed):
    inp = _inputs(case, seed)
    if case["kind"] == "batch":
        return dict(kind="batch", probs=[P.Problem(*p) for p in inp],
                    params=P.make_params(eta=case["eta"], max_iter=case["iters"]))
    if case["kind"] == "cost":
        return dict(kind="solve", prob=P.Problem.from_cost(*inp),
                    params=P.make_params(eta=case["eta"], max_iter=case["iters"]))
    if case["kind"] == "grad":
        return dict(kind="grad", inp=inp, case=case)
    prob = P.Problem(*inp[:4], metric=case["metric"])
    if case["kind"] == "solve":
        return dict(kind="solve", prob=prob,
                    params=P.make_params(eta=case["eta"], max_iter=case["iters"], precision=case["precision"]))
    # a loop over steps and a certificate after a solve know the cost's scale
    prob.cost_scale, _ = P.cost_scale(prob)
    prob.cost_norm = 1.0
    state = P.State(inp[4], inp[5], case["t"], _lam(case["eta"], case["t"]), 0.0)
    return dict(kind=case["kind"], prob=prob, state=state,
                params=P.make_params(eta=case["eta"], precision=case["precision"]))


# ------------------------------------------------------------------ one pass

def run(state):
    kind = state["kind"]
    if kind == "solve":
        s, rep, _ = P.solve(state["prob"], state["params"])
        return dict(nu=s.nu, theta=s.theta, iters=rep["iters"], res=rep["final_res"])
    if kind == "step":
        s = state["state"].clone()
        res, _ = P.step(state["prob"], state["params"], s)
        return dict(nu=s.nu, theta=s.theta, res=res)
    if kind == "batch":
        states, reps, _ = P.solve_batched(state["probs"], state["params"])
        return dict(nu=torch.cat([s.nu for s in states]), theta=torch.cat([s.theta for s in states]),
                    iters=sum(r["iters"] for r in reps))
    if kind == "cert":
        return P.certificate(state["prob"], state["params"], state["state"])
    x, y, r, c = state["inp"]
    x, y = x.detach().requires_grad_(), y.detach().requires_grad_()
    case = state["case"]
    cost = P.LampOT.apply(x, y, r, c, case["eta"], 0.0, case["iters"], 0.0, case["metric"])
    cost.backward()
    return dict(cost=cost.detach(), gx=x.grad, gy=y.grad)


# ------------------------------------------------------------------ what a pass cannot do without

def work(case):
    """Per pair of a sweep and coupling: one exponential, its argument and its sum; per pair of a
    sweep the inner product (or the matrix entry).  Bytes: inputs read once, results written once; a
    cost matrix once per sweep (the column sums need every row's normaliser)."""
    kind = case["kind"]
    if kind == "batch":
        sizes = _batch_sizes(case)
        return dict(flops=case["iters"] * 2.0 * sum(n * m * (2 * d + 8) for n, m, d in sizes),
                    bytes=sum((n + m) * (4.0 * d + 8) + 16.0 * m for n, m, d in sizes))
    n, m = case["n"], case["m"]
    if kind == "cost":
        b = 4 if case["dtype"] == "float32" else 2
        return dict(flops=case["iters"] * 2.0 * n * m * 9, bytes=case["iters"] * 2.0 * n * m * b + 8.0 * (n + 3 * m))
    d = case["d"]
    pts = (n + m) * (4.0 * d + 8)
    sweep = 2.0 * d + 8
    if kind == "cert":            # normalisers, column residual, costs and dual values, two rounding passes
        return dict(flops=1.0 * n * m * 5 * sweep, bytes=pts + 16.0 * m)
    if kind == "step":
        return dict(flops=1.0 * n * m * 2 * sweep, bytes=pts + 32.0 * m)
    flops = case["iters"] * 2.0 * n * m * sweep
    if kind == "grad":            # cost and two gradients beside the iterations
        return dict(flops=flops + 3.0 * n * m * (4 * d + 5), bytes=pts * 2)
    return dict(flops=flops, bytes=pts + 16.0 * m)


# ------------------------------------------------------------------ FP64 reference

class _Exact:
    """Algorithm 2 of the paper in FP64, the cost evaluated in row chunks."""

    def __init__(self, r, c, x=None, y=None, metric="sqeuclid", cost=None, rounded=None):
        self.r, self.c, self.metric, self.cost = r, c, metric, cost
        self.n, self.m = r.numel(), c.numel()
        if cost is None:
            mu = 0.5 * (x[0].double() + y[0].double())
            self.x, self.y = x.double() - mu, y.double() - mu
            self.x2, self.y2 = self.x.square().sum(1), self.y.square().sum(1)
            # a precision form solves the problem whose inner products take rounded centred points
            self.xr, self.yr = (self.x, self.y) if rounded is None else (self.x.to(rounded).double(), self.y.to(rounded).double())
        self.step_rows = max(1, min(self.n, int(2 ** 27 // self.m)))
        self.s = 1.0
        self.s = 1.0 / max(float(self.dist(a, b, full=True).max()) for a, b in self.chunks())

    def chunks(self):
        for a in range(0, self.n, self.step_rows):
            yield a, min(self.n, a + self.step_rows)

    def dist(self, a, b, full=False):
        """s * the ground cost of rows a..b (full: the unrounded points, for the scale)."""
        if self.cost is not None:
            return self.cost[a:b].double().mul_(self.s)
        if self.metric == "sqeuclid":
            u, v = (self.x, self.y) if full else (self.xr, self.yr)
            out = torch.addmm(self.y2[None, :], u[a:b], v.t(), alpha=-2.0).add_(self.x2[a:b, None])
            return out.mul_(self.s)
        out = None
        for k in range(self.x.shape[1]):
            t = (self.x[a:b, k, None] - self.y[None, :, k]).abs_()
            out = t if out is None else (out.add_(t) if self.metric == "l1" else torch.maximum(out, t, out=out))
        return out.mul_(self.s)

    def coupling(self, C, lam, v):
        """log p of the rows: -lam (C + 2 v) minus its row log-sum-exp, and that."""
        e = torch.add(C, v[None, :], alpha=2.0).mul_(-lam)
        mx = e.amax(1, keepdim=True)
        e.sub_(mx)
        z = torch.exp(e).sum(1, keepdim=True).log_()
        return e.sub_(z), (z + mx)[:, 0]

    def step(self, nu, theta, lam, eta, tau1=0.5, alpha=0.01, beta=1.1):
        lam1 = tau1 + lam * (1.0 - tau1 * eta)
        w = tau1 / lam1
        nubar = nu + w * (theta - nu)
        colA, colB = torch.zeros_like(nu), torch.zeros_like(nu)
        for a, b in self.chunks():
            C = self.dist(a, b)
            for col, l, v in ((colA, lam, nu), (colB, lam1, nubar)):
                e, _ = self.coupling(C, l, v)
                col += self.r[a:b] @ e.exp_()
        ca = self.c + alpha / self.m
        at = torch.atanh(theta)
        tbar, that = torch.tanh(at + (colA - self.c) / ca), torch.tanh(at + (colB - self.c) / ca)
        res = float((colA - self.c).abs().sum())
        clip = math.tanh(beta / 2.0)
        return nu + w * (tbar - nu), that.clamp(-clip, clip), lam1, res

    def solve(self, eta, iters):
        nu = torch.zeros(self.m, dtype=torch.float64, device="cuda")
        theta, lam, res = nu.clone(), 0.0, 0.0
        for _ in range(iters):
            nu, theta, lam, res = self.step(nu, theta, lam, eta)
        return nu, theta, lam, res


def _seconds(case):
    """About how long the FP64 reference of a case takes on the GPU."""
    if case["kind"] == "batch":
        return case["iters"] * sum(1e-3 + n * m * 6e-11 for n, m, _ in _batch_sizes(case))
    per = 6e-11 if case.get("metric", "sqeuclid") == "sqeuclid" else 5e-11 + 1.5e-11 * case["d"]
    return case["n"] * case["m"] * per * (case.get("iters", 1) + 2) * (2 if case["kind"] == "grad" else 1)


def exact(case, seed):
    if _seconds(case) > 15.0:
        return None
    inp = _inputs(case, seed)
    kind = case["kind"]
    if kind == "batch":
        got = [_Exact(r, c, x, y).solve(case["eta"], case["iters"]) for x, y, r, c in inp]
        return dict(nu=torch.cat([g[0] for g in got]), theta=torch.cat([g[1] for g in got]),
                    iters=case["iters"] * case["count"])
    if kind == "cost":
        nu, theta, _, res = _Exact(inp[1], inp[2], cost=inp[0]).solve(case["eta"], case["iters"])
        return dict(nu=nu, theta=theta, iters=case["iters"], res=res)
    x, y, r, c = inp[:4]
    rounded = {"bf16_mfma": torch.bfloat16, "fp16_mfma": torch.float16, "fp32_mfma": torch.float32}.get(case.get("precision"))
    ex = _Exact(r, c, x, y, case["metric"], rounded=rounded)
    if kind == "solve":
        nu, theta, _, res = ex.solve(case["eta"], case["iters"])
        return dict(nu=nu, theta=theta, iters=case["iters"], res=res)
    if kind == "step":
        nu, theta, _, res = ex.step(inp[4], inp[5], _lam(case["eta"], case["t"]), case["eta"])
        return dict(nu=nu, theta=theta, res=res)
    if kind == "cert":
        return _exact_cert(ex, case, inp[4], inp[5])
    nu, _, lam, _ = ex.solve(case["eta"], case["iters"])
    cost = torch.zeros((), dtype=torch.float64, device="cuda")
    gx, gy = torch.zeros_like(ex.x), torch.zeros_like(ex.y)
    for a, b in ex.chunks():
        C = ex.dist(a, b)
        e, _ = ex.coupling(C, lam, nu)
        X = e.exp_().mul_(r[a:b, None])
        cost += (X * C).sum()
        if ex.metric == "sqeuclid":
            gx[a:b] = 2 * ex.s * (X.sum(1)[:, None] * ex.x[a:b] - X @ ex.y)
            gy += 2 * ex.s * (X.sum(0)[:, None] * ex.y - X.t().contiguous() @ ex.x[a:b])
            continue
        diff = [ex.x[a:b, k, None] - ex.y[None, :, k] for k in range(ex.x.shape[1])]
        if ex.metric == "linf":
            top = torch.stack([t.abs() for t in diff]).argmax(0)
        for k, t in enumerate(diff):
            G = ex.s * X * t.sign()
            if ex.metric == "linf":
                G = G * (top == k)
            gx[a:b, k] = G.sum(1)
            gy[:, k] -= G.sum(0)
    return dict(cost=cost, gx=gx, gy=gy)


def _exact_cert(ex, case, nu, theta):
    lam, eta, r, c = _lam(case["eta"], case["t"]), case["eta"], ex.r, ex.c
    n = ex.n
    cost, col, duals = 0.0, torch.zeros_like(nu), [0.0] * 4
    for a, b in ex.chunks():
        C = ex.dist(a, b)
        for q, v in enumerate((theta, nu)):
            t = torch.add(C, v[None, :], alpha=2.0)
            mn = t.amin(1)
            duals[q] += float(r[a:b] @ mn)
            if eta > 0:
                z = t.sub_(mn[:, None]).mul_(-1.0 / eta).exp_().sum(1)
                duals[2 + q] += float(r[a:b] @ (mn - eta * z.log()))
        p = ex.coupling(C, lam, nu)[0].exp_()
        cost += float(r[a:b] @ (p * C).sum(1))
        col += r[a:b] @ p
    y = (c / col).clamp(max=1.0)
    dc = c - y * col
    dr, kept, corr = torch.zeros(n, dtype=torch.float64, device="cuda"), 0.0, 0.0
    for a, b in ex.chunks():
        C = ex.dist(a, b)
        p = ex.coupling(C, lam, nu)[0].exp_()
        dr[a:b] = r[a:b] * (p @ (1.0 - y))
        kept += float(r[a:b] @ ((p * C) @ y))
        corr += float(dr[a:b] @ (C @ dc))
    for q, v in enumerate((theta, nu)):
        duals[q] -= 2.0 * float(c @ v)
        duals[2 + q] -= 2.0 * float(c @ v)
    res = float((col - c).abs().sum())
    top = cost + 2.0 * res
    return dict(col_res=res, cost=cost, dual_theta=duals[0], dual_nu=duals[1], primal_penalized=top,
                gap=top - max(duals[0], duals[1]), prop_bound=4.0 * res + 2.0 * math.log(ex.m) / case["t"],
                cost_scale=ex.s, cost_norm=1.0, t=case["t"], rounded_cost=kept + corr / float(dr.sum()),
                dual_eta_theta=duals[2] if eta > 0 else None, dual_eta_nu=duals[3] if eta > 0 else None,
                row_res=None, dt=None, midpoint_bound=None)
