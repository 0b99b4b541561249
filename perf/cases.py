"""The calls that this library's users wait for, as cases that can be timed and checked.

The path is a regression of Y on the columns of X (N rows, d columns): sketch
[X|Y], factor the Hessian sketch, iterate on residual gradients, and
differentiate the solution.  Each case is one call of a public entry point of
`paper_2509_06856_amd.slse` on data resident on the GPU, from the smallest
problem of the benchmark and the tests (16384 x 32) to its largest
(2^22 x 512), with row and column counts that are no powers of 2 among them.

A case is a dict of plain values:
  op      grad (fused residual gradient), sketch, factor, solve, train
          (forward and backward of the differentiable solve), batched
  N, d    rows and columns; rows: rows of the matrix that is factored
  dtype   f32 or f64 storage; residuals and solutions are float64 always
and per op the options named in `listed`.
"""
import math
import random

import torch

from paper_2509_06856_amd import slse as G

DTYPE = {"f32": torch.float32, "f64": torch.float64}


def listed():
    return [
        # One gradient of the small benchmark problem: a caller with an iteration of its
        # own, where the call's latency is all there is.
        dict(name="grad_small_f64", op="grad", N=16384, d=32, dtype="f64", pad=0),
        # The same call on a table as it comes: a million rows of 100 features and an
        # intercept, whose rows start at no vector boundary.
        dict(name="grad_ragged_f32", op="grad", N=1000003, d=101, dtype="f32", pad=0),
        # The SRHT of the largest benchmark problem: one level of N/2 rows and the Hessian
        # sketch of 6d rows, in float32.
        dict(name="srht_f32", op="sketch", kind="srht", N=1 << 22, d=512, dtype="f32", levels=1, bf16=False),
        # The CountSketch with every nested level, on the experiments' float64 problem.
        dict(name="countsketch_f64", op="sketch", kind="countsketch", N=1 << 20, d=64, dtype="f64", levels=0,
             bf16=False),
        # The Gaussian sketch of float32 data on the matrix cores (the caller's choice).
        dict(name="gauss_bf16", op="sketch", kind="gaussian", N=1 << 20, d=256, dtype="f32", levels=1, bf16=True),
        # The Gaussian sketch in the data's own precision, as a float64 solve takes it.
        dict(name="gauss_f64", op="sketch", kind="gaussian", N=1 << 17, d=64, dtype="f64", levels=2, bf16=False),
        # Factor and preconditioner of the largest Hessian sketch, through its Gram matrix.
        dict(name="factor_chol_f32", op="factor", method="chol", rows=3072, d=512, dtype="f32", kappa=1e3),
        # The same of an ill-conditioned sketch, through CholeskyQR3.
        dict(name="factor_qr_f64", op="factor", method="qr", rows=1536, d=256, dtype="f64", kappa=1e8),
        # A whole solve of the small problem with the call's defaults (no graph, with its
        # report): an interactive fit.
        dict(name="solve_small_f64", op="solve", kind="srht", N=16384, d=32, dtype="f64", factor="chol", kappa=1.0,
             steps=30, graph=False),
        # A whole solve of the largest problem in mixed precision, replayed from its graph:
        # the benchmark's headline.
        dict(name="solve_mixed_f32", op="solve", kind="srht", N=1 << 22, d=512, dtype="f32", factor="chol",
             kappa=1e6, steps=26, graph=True),
        # A least-squares layer inside a differentiable program: the solution and the
        # gradients of X and Y.
        dict(name="train_f32", op="train", kind="srht", N=1 << 20, d=256, dtype="f32", factor="chol", kappa=1.0,
             steps=24),
        # 64 heavy-tailed regressions of uneven size at once.
        dict(name="batched_f32", op="batched", B=64, n_lo=1 << 14, n_hi=1 << 18, dtype="f32", steps=30),
    ]


def _log_int(rng, lo, hi):
    """A whole number spread evenly over the logarithm of [lo, hi]; one in four a power of 2."""
    v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    v = min(max(v, lo), hi)
    if rng.random() < 0.25:
        p = 1 << int(math.floor(math.log2(v)))
        v = p if p >= lo else v
    return v


def draw(rng):
    op = rng.choice(["grad", "grad", "srht", "countsketch", "gaussian", "gaussian", "factor", "factor", "solve",
                     "solve", "train", "batched"])
    dtype = rng.choice(["f32", "f64"])
    wide = 1 if dtype == "f32" else 2
    d = _log_int(rng, 16, 512)
    if op == "grad":
        return dict(op="grad", N=_log_int(rng, 4096, min(1 << 22, (1 << 30) // (d * wide))), d=d, dtype=dtype,
                    pad=rng.choice([0, 0, 1, 4, 31]))
    if op in ("srht", "countsketch"):
        return dict(op="sketch", kind=op, N=_log_int(rng, 64 * d, min(1 << 22, (1 << 30) // (d * wide))), d=d,
                    dtype=dtype, levels=rng.choice([0, 1]) if op == "srht" else 0, bf16=False)
    if op == "gaussian":
        bf16 = dtype == "f32" and rng.random() < 0.5
        d = _log_int(rng, 16, 256)
        most = (1 << 36 if bf16 else 1 << 30) // (d * d)
        return dict(op="sketch", kind="gaussian", N=_log_int(rng, 2048, min(1 << 20, max(4096, most))), d=d,
                    dtype=dtype, levels=rng.choice([1, 2]), bf16=bf16)
    if op == "factor":
        method = rng.choice(["chol", "qr"])
        return dict(op="factor", method=method, rows=d * rng.choice([2, 3, 6, 12]) + rng.choice([0, 1, 17]), d=d,
                    dtype="f64" if method == "qr" else dtype,
                    kappa=10.0 ** rng.uniform(4, 10) if method == "qr" else 10.0 ** rng.uniform(0, 3))
    if op == "batched":
        n_lo = 1 << 14
        return dict(op="batched", B=_log_int(rng, 4, 64), n_lo=n_lo, n_hi=_log_int(rng, n_lo, 1 << 17), dtype=dtype,
                    steps=rng.randint(20, 40))
    d = _log_int(rng, 16, 256)
    N = _log_int(rng, 64 * d, min(1 << 22, (1 << 29) // (d * wide)))
    if op == "train":
        return dict(op="train", kind="srht", N=min(N, 1 << 20), d=d, dtype=dtype, factor="chol",
                    kappa=10.0 ** rng.uniform(0, 2), steps=24)
    return dict(op="solve", kind=rng.choice(["srht", "srht", "countsketch"]), N=N, d=d, dtype=dtype,
                factor=rng.choice(["chol", "chol", "qr"]), kappa=10.0 ** rng.uniform(0, 4),
                steps=rng.randint(24, 30), graph=rng.random() < 0.5)


def _levels(case):
    """The nested sketch sizes of a sketch or a solve: the experiments' schedule (8d, doubling
    to N/2), its largest level alone, or, for the Gaussian sketch, its first levels."""
    N, d, n = case["N"], case["d"], case.get("levels", 0)
    if case["kind"] == "gaussian":
        return [6 * d] if n == 1 else [8 * d << i for i in range(n)]
    m = G.paper_schedule(N, d)
    return m[-1:] if n == 1 else m


def _regression(g, N, d, dt, kappa, sigma=1e-2):
    """X = Z diag(s) with s log-spaced over 1..1/kappa (the experiments' recipe), Y = X beta + noise."""
    X = torch.randn(N, d, generator=g, device="cuda", dtype=dt)
    if kappa > 1:
        X *= torch.logspace(0, -math.log10(kappa), d, device="cuda", dtype=torch.float64).to(dt)
    beta = torch.randn(d, generator=g, device="cuda", dtype=torch.float64)
    Y = torch.mv(X, beta.to(dt)) + sigma * torch.randn(N, generator=g, device="cuda", dtype=dt)
    return X, Y, beta


def _batch_shapes(case):
    """The (N_b, d_b) of a batch: N_b uniform in [n_lo, n_hi], d_b one of five widths."""
    rng = random.Random(case["B"])
    return [(rng.randint(case["n_lo"], case["n_hi"]), rng.choice((16, 32, 64, 128, 256)))
            for _ in range(case["B"])]


def _batch(case, g):
    """B regressions with Student-t(3) rows and unit columns."""
    dt, out = DTYPE[case["dtype"]], []
    for n, d in _batch_shapes(case):
        X = torch.randn(n, d, generator=g, device="cuda", dtype=dt)
        X /= (torch.randn(n, 3, generator=g, device="cuda", dtype=dt).square().sum(1, keepdim=True) / 3).sqrt()
        X /= X.double().square().sum(0).sqrt().to(dt)
        beta = torch.randn(d, generator=g, device="cuda", dtype=dt)
        out.append((X, torch.mv(X, beta) + 1e-2 * torch.randn(n, generator=g, device="cuda", dtype=dt)))
    return out


def _params(case, N, d, seed, m=None, **kw):
    m = G.paper_schedule(N, d) if m is None else m
    return G.Params(kind=case.get("kind", "srht"), seed=seed, m=m, a=[2] * len(m), r=6 * d, s_max=case["steps"],
                    precision="mixed" if case["dtype"] == "f32" else "f64", factor=case.get("factor", "chol"), **kw)


def prepare(case, seed):
    """Data as a program has them, and the parameters that it keeps; `seed` keys the data and the sketch."""
    op, dt = case["op"], DTYPE[case["dtype"]]
    g = torch.Generator(device="cuda").manual_seed(seed)
    if op == "batched":
        data = _batch(case, g)
        ps = [_params(case, *X.shape, seed + 100 * b) for b, (X, _) in enumerate(data)]
        return dict(op=op, Xs=[X for X, _ in data], Ys=[Y for _, Y in data], params=ps)
    if op == "factor":
        A, _, _ = _regression(g, case["rows"], case["d"], dt, case["kappa"])
        return dict(op=op, A=A, d=case["d"], scale=1.0 / case["rows"], method=case["method"])
    N, d = case["N"], case["d"]
    X, Y, beta = _regression(g, N, d, dt, case.get("kappa", 1.0))
    if op == "grad":
        if case["pad"]:  # the first d columns of a wider table
            table = torch.empty(N, d + case["pad"], device="cuda", dtype=dt)
            table[:, :d] = X
            X = table[:, :d]
        beta += 1e-2 * torch.randn(d, generator=g, device="cuda", dtype=torch.float64)
        return dict(op=op, X=X, Y=Y, beta=beta, scale=1.0 / N)
    if op == "sketch":
        return dict(op=op, X=X, Y=Y, kind=case["kind"], seed=seed, m=_levels(case), r=6 * d, bf16=case["bf16"])
    st = dict(op=op, X=X, Y=Y, params=_params(case, N, d, seed, use_graph=case.get("graph", False)),
              report=not case.get("graph", False))
    if op == "train":
        st["X"].requires_grad_()
        st["Y"].requires_grad_()
        st["w"] = torch.randn(d, generator=g, device="cuda", dtype=torch.float64)
    return st


def run(state):
    op = state["op"]
    if op == "grad":
        return G.fused_resid_grad(state["X"], state["Y"], state["beta"], scale=state["scale"])
    if op == "sketch":
        return G.sketch_apply(state["X"], state["Y"], state["kind"], state["seed"], state["m"], state["r"],
                              bf16=state["bf16"])[:2]
    if op == "factor":
        return G.factor(state["A"], state["d"], state["scale"], state["method"])
    if op == "solve":
        return G.solve(state["X"], state["Y"], state["params"], report=state["report"])[0]
    if op == "train":
        beta = G.SLSEFunction.apply(state["X"], state["Y"], state["params"])
        return (beta.detach(), *torch.autograd.grad(beta, (state["X"], state["Y"]), state["w"]))
    return G.solve_batched(state["Xs"], state["Ys"], state["params"], report=False)[0]


def _solve_work(N, d, m, steps, es):
    """A solve's necessary passes: the data once for the sketch, twice each level, once a step.
    Steps depend on each other, and data over the chip's caches have to be read again for each."""
    rows = N + 2 * sum(m) + steps * N
    return rows * (d + 1) * es, 4.0 * (rows - N) * d


def work(case):
    es = 4 if case["dtype"] == "f32" else 8
    op = case["op"]
    if op == "batched":
        each = [_solve_work(N, d, G.paper_schedule(N, d), case["steps"], es) for N, d in _batch_shapes(case)]
        return {"bytes": sum(b for b, _ in each), "flops": sum(f for _, f in each)}
    d = case["d"]
    if op == "factor":
        passes = 1 if case["method"] == "chol" else 3
        return {"bytes": case["rows"] * d * es + 2 * 8 * d * d,
                "flops": passes * (case["rows"] * d * d + d ** 3 / 3) + d ** 3}
    N = case["N"]
    row = (d + 1) * es
    if op == "grad":
        return {"bytes": N * row + 16 * d, "flops": 4.0 * N * d}
    if op == "sketch":
        m, r = _levels(case), 6 * d
        rows = sum(m) if case["kind"] == "countsketch" else m[-1]
        flops = {"srht": N * math.log2(N), "countsketch": 4.0 * N, "gaussian": 2.0 * N * (m[-1] + r)}[case["kind"]]
        return {"bytes": (N + rows + r) * row, "flops": flops * (d + 1)}
    b, f = _solve_work(N, d, G.paper_schedule(N, d), case["steps"], es)
    if op == "train":
        return {"bytes": b + (case["steps"] + 2) * N * row, "flops": f + 4.0 * N * d * (case["steps"] + 2)}
    return {"bytes": b, "flops": f}


# The same results in 64 bits, without the library: the random streams of the sketches are
# Philox4x64-10 (Salmon et al., 2011) keyed by (seed, stream), here on int64 tensors.
_M = (0xD2E7470EE14C6C93, 0xCA5A826395121157)
_W = (0x9E3779B97F4A7C15, 0xBB67AE8584CAA73B)
_LOW = 0xFFFFFFFF


def _i64(v):
    v &= (1 << 64) - 1
    return v - (1 << 64) if v >> 63 else v


def _mulhi(a, x):
    """The upper words of a * x, both unsigned."""
    a0, a1, x0, x1 = a & _LOW, a >> 32, x & _LOW, (x >> 32) & _LOW
    low = a0 * x1 + (((a0 * x0) >> 32) & _LOW)
    mid = a1 * x0 + (low & _LOW)
    return a1 * x1 + ((low >> 32) & _LOW) + ((mid >> 32) & _LOW)


def _philox(c0, c1, seed, stream):
    zero = torch.zeros_like(c0)
    x, k = [c0, c1 + zero, zero, zero], [seed, stream]
    for _ in range(10):
        h0, l0 = _mulhi(_M[0], x[0]), x[0] * _i64(_M[0])
        h1, l1 = _mulhi(_M[1], x[2]), x[2] * _i64(_M[1])
        x = [h1 ^ x[1] ^ _i64(k[0]), l1, h0 ^ x[3] ^ _i64(k[1]), l0]
        k = [k[0] + _W[0], k[1] + _W[1]]
    return x


def _permute(x, seed, stream, p):
    """The keyed permutation of [0, 2^p): four Feistel rounds on halves of ceil(p/2) bits, walked
    until the image lies inside."""
    h = (p + 1) // 2
    y, out = x, torch.ones_like(x, dtype=torch.bool)
    while bool(out.any()):
        left, right = y[out] >> h, y[out] & ((1 << h) - 1)
        for i in range(4):
            f = _philox(right, torch.full_like(right, i), seed, stream)[0] & ((1 << h) - 1)
            left, right = right, left ^ f
        y = y.clone()
        y[out] = (left << h) | right
        out = y >= 1 << p
    return y


def _signs(bit):
    return 1.0 - 2.0 * (bit & 1).double()


def _exact_sketch(st, case):
    N, d, seed, m, r = case["N"], case["d"], st["seed"], st["m"], st["r"]
    W = torch.cat([st["X"], st["Y"][:, None]], 1)
    j = torch.arange(N, device="cuda")
    if case["kind"] == "srht":
        p = max(1, (N - 1).bit_length())
        j = torch.arange(1 << p, device="cuda")
        src = _permute(j, seed, 2, p)
        words = torch.stack(_philox(j[: max(1, len(j) >> 8)], j[:1] * 0, seed, 1), 1)
        sign = _signs(words[j >> 8, (j >> 6) & 3] >> (j & 63))
        orders = [_permute(j[:n], seed, s, p) for n, s in ((m[-1], 3), (r, 4))]
        outs = [torch.empty(len(o), d + 1, device="cuda", dtype=torch.float64) for o in orders]
        for c in range(0, d + 1, 64):  # some columns at a time
            V = torch.zeros(1 << p, min(64, d + 1 - c), device="cuda", dtype=torch.float64)
            V[src < N] = W[src[src < N], c:c + 64].double()
            V *= sign[:, None]
            for b in range(p):
                v = V.view(-1, 2, 1 << b, V.shape[1])
                V = torch.stack([v[:, 0] + v[:, 1], v[:, 0] - v[:, 1]], 1).view(1 << p, -1)
            for o, out in zip(orders, outs):
                out[:, c:c + 64] = V[o]
        return tuple(outs)
    if case["kind"] == "countsketch":
        w = _philox(j, j[:1] * 0, seed, 5)
        SW, A = W.double() * _signs(w[1])[:, None], []
        for n in m:
            A.append(torch.zeros(n, d + 1, device="cuda", dtype=torch.float64).index_add_(0, w[0] & (n - 1), SW))
        w = _philox(j, j[:1] * 0, seed, 6)
        bucket = (((w[0] >> 32) & _LOW) * r) >> 32
        hat = torch.zeros(r, d + 1, device="cuda", dtype=torch.float64)
        return torch.cat(A), hat.index_add_(0, bucket, W.double() * _signs(w[1])[:, None])
    low = (lambda t: t.float().bfloat16().double()) if case["bf16"] else (lambda t: t.double())
    outs = []
    for rows, stream in ((m[-1], 7), (r, 8)):
        blocks = torch.arange((rows + 7) // 8, device="cuda")
        out = torch.zeros(rows, d + 1, device="cuda", dtype=torch.float64)
        step = max(1, (1 << 22) // len(blocks))
        for a in range(0, N, step):  # a slab of data rows at a time
            jj = j[a:a + step]
            c0, c1 = (t.reshape(-1) for t in torch.meshgrid(jj, blocks, indexing="ij"))
            words = torch.stack(_philox(c0, c1, seed, stream), 1)
            u1 = ((words & _LOW).double() + 0.5) * 2.0 ** -32
            u2 = (((words >> 32) & _LOW).double() + 0.5) * 2.0 ** -32
            rad, ang = (-2.0 * u1.log()).sqrt(), 2 * math.pi * u2
            entries = torch.stack([rad * ang.cos(), rad * ang.sin()], 2).view(len(jj), -1)[:, :rows]
            out += low(entries).T.contiguous() @ low(W[a:a + step])
        outs.append(out)
    return tuple(outs)


def _normal_solver(X):
    """b -> (X^T X)^{-1} b in float64, refined, for columns of any scale."""
    s = X.square().sum(0).sqrt()
    L = torch.linalg.cholesky((X / s).T @ (X / s))

    def solve(b):
        v = torch.cholesky_solve((b / s)[:, None], L)[:, 0] / s
        for _ in range(3):
            v = v + torch.cholesky_solve(((b - X.T @ (X @ v)) / s)[:, None], L)[:, 0] / s
        return v
    return solve, lambda r: torch.cholesky_solve(((X.T @ r) / s)[:, None], L)[:, 0] / s


def _ols(X, Y):
    X, Y = X.double(), Y.double()
    _, step = _normal_solver(X)
    beta = step(Y)
    for _ in range(3):
        beta = beta + step(Y - X @ beta)
    return beta


def exact(case, seed):
    st, op = prepare(case, seed), case["op"]
    if op == "batched":
        return [_ols(X, Y) for X, Y in zip(st["Xs"], st["Ys"])]
    if op == "factor":
        R = torch.linalg.qr((math.sqrt(st["scale"]) * st["A"].double()).cpu(), mode="r")[1]
        R = R * R.diagonal().sign()[:, None]
        inv = torch.linalg.solve_triangular(R, torch.eye(case["d"], dtype=torch.float64), upper=True)
        return R, inv @ inv.T
    if op == "grad":
        r = st["Y"].double() - st["X"].double() @ st["beta"]
        return st["scale"] * (st["X"].double().T @ r), st["scale"] * (r @ r)[None]
    if op == "sketch":
        return _exact_sketch(st, case)
    if op == "solve":
        return _ols(st["X"], st["Y"])
    X, Y = st["X"].detach().double(), st["Y"].detach().double()
    beta, lam = _ols(X, Y), _normal_solver(X)[0](st["w"])
    u = X @ lam
    return beta, torch.outer(Y - X @ beta, lam) - torch.outer(u, beta), u
