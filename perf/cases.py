"""The work that users of this library have it do, as cases that can be timed and compared.

A case is one call (or the short sequence of calls a program makes) through the public entry points:
prediction with a trained model, the product K_nm^T (K_nm v), and whole fits (squared loss with one or
several targets, logistic loss, sparse inputs).  Sizes are those of the workloads in `synth` and
`bench.py` where a pass of that size is short enough, and smaller problems of the same kinds elsewhere.
"""
import math

import numpy as np
import torch

import paper_2006_10350_amd as knm


def listed():
    return [
        # Serving: one small batch of rows against a small model.  Latency and launches are all there is.
        {"name": "predict-small", "op": "predict", "n": 200, "d": 8, "M": 1000, "t": 1, "kernel": "gaussian",
         "cross": "f16x3", "data": "normal"},
        # The headline product at full size: 28 features, one column (physics-like binary classification).
        {"name": "prod-mid", "op": "prod", "n": 11_000_000, "d": 28, "M": 100_000, "t": 1, "kernel": "gaussian",
         "cross": "f16x3", "data": "normal"},
        # Image-like multi-class product at full size: many features, most of them zero, ten columns.
        {"name": "prod-highdim", "op": "prod", "n": 2_000_000, "d": 784, "M": 50_000, "t": 10, "kernel": "gaussian",
         "cross": "f16x3", "data": "image"},
        # Speech-like many-class product: one column per class.
        {"name": "prod-manyclass", "op": "prod", "n": 120_000, "d": 440, "M": 20_000, "t": 144, "kernel": "gaussian",
         "cross": "f16x3", "data": "normal"},
        # A kernel of the distance, odd sizes.
        {"name": "prod-laplacian", "op": "prod", "n": 1_000_003, "d": 17, "M": 20_001, "t": 1, "kernel": "laplacian",
         "cross": "f16x3", "data": "normal"},
        # The arithmetic without range limits, odd sizes, skewed features (tabular regression).
        {"name": "prod-f32", "op": "prod", "n": 1_000_003, "d": 9, "M": 20_001, "t": 1, "kernel": "gaussian",
         "cross": "f32", "data": "tabular"},
        # Product on sparse rows (n-gram counts), everything prepared within the call.
        {"name": "prod-sparse", "op": "prod_csr", "n": 200_000, "d": 65_000_000, "M": 20_000, "t": 1, "nnz": 100,
         "skew": 2.5},
        # The smallest sensible fit: host work, launches and synchronisations.
        {"name": "fit-tiny", "op": "fit", "n": 20_000, "d": 8, "M": 1000, "t": 1, "iters": 10, "kernel": "gaussian",
         "cross": "f16x3", "data": "normal"},
        # An ordinary fit, one target: preconditioner, products and solves all count.
        {"name": "fit-mid", "op": "fit", "n": 1_000_000, "d": 28, "M": 20_000, "t": 1, "iters": 20, "kernel": "gaussian",
         "cross": "f16x3", "data": "normal"},
        # A multi-class fit on image-like rows: several right-hand sides through products, solves and CG.
        {"name": "fit-multiclass", "op": "fit", "n": 60_000, "d": 784, "M": 10_000, "t": 10, "iters": 20,
         "kernel": "gaussian", "cross": "f16x3", "data": "image"},
        # Logistic loss: the second factor is rebuilt in every Newton step, the products are weighted.
        {"name": "fit-logistic", "op": "fit_logistic", "n": 300_000, "d": 18, "M": 5000, "steps": 4, "iters": 5},
        # Fit on sparse rows.
        {"name": "fit-sparse", "op": "fit_csr", "n": 100_000, "d": 65_000_000, "M": 10_000, "t": 1, "iters": 10,
         "nnz": 100, "skew": 2.5},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _dense(rng, d_lo=6):
    """Features, columns, kernel, arithmetic and value distribution of a dense problem."""
    kernel = rng.choice(["gaussian"] * 7 + ["laplacian", "matern32", "matern52"])
    cross = rng.choice(["f16x3"] * 9 + ["f32"])
    t = 1 if rng.random() < 0.6 else _log(rng, 2, 144)
    d = _log(rng, d_lo, 784)
    kinds = ["normal"] if kernel != "gaussian" else ["normal", "tabular"] if d < 64 else ["normal", "tabular", "image"]
    return {"d": d, "t": t, "kernel": kernel, "cross": cross, "data": rng.choice(kinds)}


def draw(rng):
    op = rng.choice(["predict", "predict", "prod", "prod", "prod", "prod", "prod_csr", "fit", "fit", "fit", "fit_logistic",
                     "fit_csr"])
    if op == "predict":
        case = {"op": op, "n": _log(rng, 1, 50_000), "M": _log(rng, 300, 50_000), **_dense(rng)}
    elif op == "prod":
        case = {"op": op, "n": _log(rng, 5000, 11_000_000), "M": _log(rng, 500, 100_000), **_dense(rng)}
    elif op == "fit":
        case = {"op": op, "n": _log(rng, 5000, 1_000_000), "M": _log(rng, 300, 20_000), "iters": rng.randint(5, 20),
                **_dense(rng, 10)}
        case["t"] = min(case["t"], 16)
    elif op == "fit_logistic":
        case = {"op": op, "n": _log(rng, 5000, 300_000), "d": _log(rng, 10, 44), "M": _log(rng, 300, 5000),
                "steps": rng.randint(2, 4), "iters": rng.randint(3, 5)}
    else:
        case = {"op": op, "n": _log(rng, 5000, 200_000), "d": _log(rng, 100_000, 65_000_000), "M": _log(rng, 500, 20_000),
                "t": 1, "nnz": rng.randint(30, 100), "skew": 2.5}
        if op == "fit_csr":
            case["n"], case["M"], case["iters"] = min(case["n"], 100_000), min(case["M"], 10_000), rng.randint(5, 10)
    if op != "predict":
        case["M"] = min(case["M"], case["n"] // 4)
    if op in ("prod", "fit"):
        # no more kernel work than the full-size product with many features
        dear = (3.5 if case["cross"] == "f32" else 1.0) * (2.0 if case["kernel"] != "gaussian" else 1.0)
        per_entry = dear * (30.0 + case["d"] + 4.0 * case["t"]) * (case.get("iters", 0) + 1)
        case["n"] = max(case["M"], min(case["n"], int(6.0e13 / per_entry / case["M"])))
    return case


# ---- inputs -----------------------------------------------------------------------------------------

_contexts = {}


def _context(kernel="gaussian", cross="f16x3"):
    """A program makes its context once and keeps it."""
    key = (torch.cuda.current_device(), kernel, cross)
    if key not in _contexts:
        ctx = knm.Context()
        ctx.set_kernel(kernel)
        ctx.set_cross_term(cross)
        _contexts[key] = ctx
    return _contexts[key]


def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _rows(n, d, data, g):
    """Standardised rows: normal features; half of them skewed (lognormal) and half whole-valued; or
    image-like rows with four fifths exact zeros."""
    X = torch.empty(n, d, device="cuda", dtype=torch.float32)
    step = max(1, (1 << 27) // d)
    for lo in range(0, n, step):
        x = X[lo:lo + step]
        if data == "normal":
            x.normal_(generator=g)
        elif data == "tabular":
            h = d // 2
            whole = torch.randint(0, 25, (x.shape[0], h), generator=g, device="cuda").float()
            x[:, :h] = (whole - 12.0) / math.sqrt(52.0)
            skewed = torch.randn(x.shape[0], d - h, generator=g, device="cuda").exp()
            x[:, h:] = (skewed - math.exp(0.5)) / math.sqrt((math.e - 1.0) * math.e)
        else:
            x.uniform_(generator=g)
            x.mul_(torch.rand(x.shape, generator=g, device="cuda") < 0.2)
    return X


def _sigma(d, data):
    """Length scale of the order of the distances, as the workloads have it."""
    return {"image": 0.45, "normal": 0.75, "tabular": 0.4}[data] * math.sqrt(d)


def _targets(X, t, g):
    """+-1 for one target (a noisy nonlinear rule), one-hot rows for several (nearest of t prototypes)."""
    n, d = X.shape
    if t == 1:
        a, b = torch.randn(2, d, 1, generator=g, device="cuda")
        score = (X @ a + (X @ b) * torch.tanh(X @ a / math.sqrt(d))) / math.sqrt(d)
        score += 0.3 * torch.randn(n, 1, generator=g, device="cuda")
        return torch.where(score >= score.median(), 1.0, -1.0).contiguous()
    P = X[torch.randint(0, n, (t,), generator=g, device="cuda")]
    near = ((P * P).sum(1)[None, :] - 2.0 * (X @ P.T)).argmin(1)
    return torch.nn.functional.one_hot(near, t).float()


def _sparse_rows(n, d, nnz, skew, g):
    """CSR rows like n-gram counts: lognormal row lengths, a few features in a large share of the rows."""
    lengths = torch.exp(math.log(nnz) + 0.5 * torch.randn(n, generator=g, device="cuda")).round().long()
    lengths[::97] = 0  # some empty rows
    total = int(lengths.sum())
    col = (d * torch.rand(total, generator=g, device="cuda", dtype=torch.float64).pow(skew)).long().clamp_(max=d - 1)
    row = torch.arange(n, device="cuda").repeat_interleave(lengths)
    key, count = torch.unique(row * d + col, return_counts=True)  # a feature once per row, with its count
    row, col = key // d, key % d
    crow = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    crow[1:] = torch.bincount(row, minlength=n).cumsum(0)
    return crow, col, count.float()


def _take_rows(crow, col, val, pick):
    length = crow[pick + 1] - crow[pick]
    out = torch.zeros(pick.numel() + 1, dtype=torch.int64, device="cuda")
    out[1:] = length.cumsum(0)
    at = crow[pick].repeat_interleave(length) + torch.arange(int(out[-1]), device="cuda") - out[:-1].repeat_interleave(length)
    return out, col[at], val[at]


def prepare(case, seed):
    g = _generator(seed)
    op, n, d, M = case["op"], case["n"], case["d"], case["M"]
    s = {"op": op, "case": case}
    if op in ("prod_csr", "fit_csr"):
        crow, col, val = _sparse_rows(n, d, case["nnz"], case["skew"], g)
        pick = torch.randperm(n, generator=g, device="cuda")[:M].sort().values
        s["X"] = torch.sparse_csr_tensor(crow, col, val, size=(n, d), check_invariants=False)
        s["C"] = torch.sparse_csr_tensor(*_take_rows(crow, col, val, pick), size=(M, d), check_invariants=False)
        s["sigma"], s["ctx"] = math.sqrt(case["nnz"]), _context()
        if op == "prod_csr":
            s["V"] = torch.randn(M, case["t"], generator=g, device="cuda")
        else:
            row = torch.arange(n, device="cuda").repeat_interleave(crow[1:] - crow[:-1])
            weight = torch.randn(1 << 16, generator=g, device="cuda")[col % (1 << 16)]
            score = torch.zeros(n, device="cuda", dtype=torch.float64).index_add_(0, row, (val * weight).double())
            s["Y"] = torch.tanh(0.05 * score).float().reshape(n, 1)
        return s
    data = case.get("data", "normal")
    s["sigma"] = _sigma(d, data)
    s["ctx"] = _context(case.get("kernel", "gaussian"), case.get("cross", "f16x3"))
    if op == "predict":
        s["X"], s["C"] = _rows(n, d, data, g), _rows(M, d, data, g)
        s["alpha"] = torch.randn(M, case["t"], generator=g, device="cuda")
        return s
    s["X"] = _rows(n, d, data, g)
    pick = torch.randperm(n, generator=g, device="cuda")[:M]
    s["C"] = s["X"][pick].contiguous()
    if op == "prod":
        s["V"] = torch.randn(M, case["t"], generator=g, device="cuda")
        return s
    s["Y"] = _targets(s["X"], case.get("t", 1), g)
    s["Xtest"] = _rows(2000, d, data, g)
    if op == "fit_logistic":
        s["YC"] = s["Y"][pick].contiguous()
    return s


# regularised well enough for the coefficients themselves to be determined by fp32 products
LAMBDA, JITTER = 1e-5, 1e-4


def run(s):
    op, X, C, sigma, ctx, case = s["op"], s["X"], s["C"], s["sigma"], s["ctx"], s["case"]
    if op == "predict":
        return knm.falkon_predict(X, C, sigma, s["alpha"], ctx=ctx)
    if op == "prod":
        return knm.knm_prod(X, C, sigma, s["V"], ctx=ctx)
    if op == "prod_csr":
        return knm.knm_prod_csr(X, C, sigma, s["V"], ctx=ctx)
    if op == "fit":
        alpha = knm.falkon_fit(X, s["Y"], C, sigma, LAMBDA, case["iters"], JITTER, ctx=ctx)
        return {"alpha": alpha, "predicted": knm.falkon_predict(s["Xtest"], C, sigma, alpha, ctx=ctx)}
    if op == "fit_logistic":
        lambdas = [max(LAMBDA, LAMBDA * 10.0 ** (case["steps"] - 2 - k)) for k in range(case["steps"])]
        alpha, loss = knm.logfalkon_fit(X, s["Y"], C, s["YC"], sigma, lambdas, [case["iters"]] * case["steps"], JITTER,
                                        return_loss=True, ctx=ctx)
        return {"alpha": alpha, "loss": loss, "predicted": knm.falkon_predict(s["Xtest"], C, sigma, alpha, ctx=ctx)}
    return knm.falkon_fit_csr(X, s["Y"], C, sigma, LAMBDA, case["iters"], JITTER, ctx=ctx)


# ---- what a pass cannot do without ------------------------------------------------------------------


def _sharing_pairs(case):
    """Expected number of (row, centre, shared feature) triples of sparse rows."""
    d, p = case["d"], 1.0 / case["skew"]
    f = np.arange(min(d, 1_000_000), dtype=np.float64)
    share = 1.0 - np.exp(-case["nnz"] * (((f + 1) / d) ** p - (f / d) ** p))
    return case["n"] * case["M"] * float((share * share).sum())


def work(case):
    """Every kernel value once (2 d flop, 2 t for each product it takes part in); the preconditioner's
    two factorisations and the product between them, M^3 flop in all; two triangular solves with each
    factor per iteration.  Inputs read once, outputs written once."""
    op, n, d, M = case["op"], case["n"], case["d"], case["M"]
    t = case.get("t", 1)
    entries = float(n) * M
    if op == "predict":
        return {"bytes": 4.0 * (n * d + M * d + M * t + n * t), "flops": entries * (2 * d + 2 * t)}
    if op == "prod":
        return {"bytes": 4.0 * (n * d + M * d + 2 * M * t), "flops": entries * (2 * d + 4 * t)}
    if op in ("prod_csr", "fit_csr"):
        nnz = case["nnz"] * (n + M)
        sweeps = 2 if op == "prod_csr" else 2 * case["iters"] + 1
        w = {"bytes": 12.0 * nnz + 8.0 * (n + M) + 8.0 * M * t, "flops": 2.0 * _sharing_pairs(case) * (1 + sweeps)}
        if op == "fit_csr":
            w["bytes"] += 4.0 * n * t
            w["flops"] += float(M) ** 3 + case["iters"] * 4.0 * M * M * t
        return w
    steps, iters = case.get("steps", 1), case["iters"]
    flops = entries * (2 * d + 2 * t * (2 * iters + 1) * steps) + steps * iters * 4.0 * M * M * t
    flops += float(M) ** 3 / 3.0 * (1 + 2 * steps) + float(M) * M * d
    return {"bytes": 4.0 * (n * d + M * d + n * t + M * t), "flops": flops}


def tolerance(case):
    """Products: fp32 data and sums.  Fits: the rounding of the fp32 products (about 3e-7) reaches the
    coefficients through T^-1, i.e. amplified by up to sqrt(1 / jitter) twice."""
    if case["op"] in ("predict", "prod", "prod_csr"):
        return {"rel": 1e-5}
    return {"rel": 1e-2, "max": 0.2}
