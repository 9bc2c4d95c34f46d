"""What rounding does to the coefficients of a fit: dense fits repeat bit for bit, and their distance from the same
iterations in 64 bits is that of the few roundings left in the solver's K^T w."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu

LAMBDA, JITTER, ITERS = 1e-5, 1e-4, 20


def _image_rows(n, d, g):
    X = torch.rand(n, d, generator=g, device="cuda")
    return X.mul_(torch.rand(n, d, generator=g, device="cuda") < 0.2)


def _kernel64(X, C, sigma):
    X, C = X.double(), C.double()
    r2 = (X * X).sum(1)[:, None] + (C * C).sum(1)[None] - 2.0 * (X @ C.T.contiguous())
    return torch.exp(-r2.clamp_min_(0.0) / (2.0 * sigma * sigma))


def _fit64(X, Y, C, sigma, round_u=False):
    """Alg. 1 in 64 bits; with round_u, K^T w is rounded to fp32 in every iteration and nothing else is."""
    n, M = X.shape[0], C.shape[0]
    K, KMM = _kernel64(X, C, sigma), _kernel64(C, C, sigma)
    KMM.fill_diagonal_(1.0 + JITTER)
    T = torch.linalg.cholesky(KMM, upper=True)
    A = torch.linalg.cholesky(T @ T.T / M + LAMBDA * torch.eye(M, device="cuda", dtype=torch.float64), upper=True)
    lower = {id(T): T.T.contiguous(), id(A): A.T.contiguous()}
    KT = K.T.contiguous()

    def solve(R, b, trans=False):
        return torch.linalg.solve_triangular(lower[id(R)] if trans else R, b, upper=not trans)

    def kt(w):
        u = KT @ w
        return u.float().double() if round_u else u

    def operator(p):
        v = solve(A, p)
        return solve(A, solve(T, kt(K @ solve(T, v)), True) + LAMBDA * n * v, True)

    r = solve(A, solve(T, kt(Y.double()), True), True)
    b, p, rho = torch.zeros_like(r), r.clone(), (r * r).sum(0)
    for _ in range(ITERS):
        q = operator(p)
        a = rho / (p * q).sum(0)
        b += a * p
        r = r - a * q
        new = (r * r).sum(0)
        p = r + new / rho * p
        rho = new
    return solve(T, solve(A, b))


# Several columns and one; classes as skewed as one-hot targets get; kernel values kept for all sweeps, whose sums are all fp64, and formed by
# every sweep of the K-loop engine (the images that the values are formed from do not fit the cap).  If every entry of K^T w is rounded to fp32
# the coefficients move by E (measured here).  The engine adds the terms of an entry in fp32 sums of 8 and those in fp64: n terms of
# size m give an rms error of m eps sqrt(n 8^2 / 3) against an entry of n m, eps that of one rounding, i.e. sqrt(64 / (3 n)) of a rounding of
# the entry, and so of E.  Sums of 64 terms would give sqrt(64^2 / (3 n)), eight times as much; the bound is 2.5 times the first.  The
# kernel values' own rounding (a few 1e-7 of random sign, averaged over the n rows) moves the coefficients by some 1e-4 times more.
@pytest.mark.parametrize("cross,t,kept", [("f16x3", 10, True), ("f16x3", 1, True), ("f32", 3, True), ("f16x3", 10, False), ("f16x3", 1, False)])
def test_coefficients_against_the_same_iterations_in_64_bits(knm, cross, t, kept):
    n, d, M = 20000, 784, 2000
    g = torch.Generator(device="cuda").manual_seed(5)
    X = _image_rows(n, d, g)
    C = X[torch.randperm(n, generator=g, device="cuda")[:M]].contiguous()
    sigma = 12.5  # exactly representable
    share = torch.tensor([0.95] + [0.05 / 9] * 9, device="cuda")
    Y = torch.nn.functional.one_hot(torch.multinomial(share, n, replacement=True, generator=g), 10).float()[:, :t].contiguous()
    ctx = knm.Context()
    ctx.set_cross_term(cross)
    if not kept:
        ctx.set_pack_limit(16 << 20)
    alpha = knm.falkon_fit(X, Y, C, sigma, LAMBDA, ITERS, JITTER, ctx=ctx)
    assert (ctx.workspace_held() > 4 * n * M) == kept, ctx.workspace_held()  # the block of the values stays with the context
    exact = _fit64(X, Y, C, sigma)
    rounded = float((_fit64(X, Y, C, sigma, round_u=True) - exact).norm() / exact.norm())
    error = float((alpha.double() - exact).norm() / exact.norm())
    print(f"\n  {cross}, t = {t}, {'kept' if kept else 'formed'}: K^T w rounded to fp32 moves the coefficients by {rounded:.2e}, the fit is {error:.2e} off")
    assert error < 2.5 * math.sqrt(64.0 / (3.0 * n)) * rounded + 1e-3


# dense fits repeat bit for bit, also after another fit has had the context's workspace in between: both engines, several columns,
# and the logistic fit (its second sweep pair is k(C, C))
def test_dense_fits_repeat_bit_for_bit(knm):
    g = torch.Generator(device="cuda").manual_seed(6)
    ctx = knm.Context()
    shapes = [(6000, 784, 700, 10), (30000, 28, 1500, 1), (9000, 60, 500, 1)]
    inputs = []
    for n, d, M, t in shapes:
        X = torch.randn(n, d, generator=g, device="cuda")
        inputs.append((X, torch.randn(n, t, generator=g, device="cuda"), X[:M].contiguous(), 0.75 * math.sqrt(d)))

    def all_fits():
        out = [knm.falkon_fit(X, Y, C, s, 1e-6, 8, 1e-8, ctx=ctx) for X, Y, C, s in inputs]
        for X, Y, C, s in inputs[1:]:
            y = torch.where(Y > 0, 1.0, -1.0)
            out.append(knm.logfalkon_fit(X, y, C, y[:C.shape[0]].contiguous(), s, [1e-4, 1e-5], [3, 3], 1e-6, ctx=ctx))
        return out

    first = all_fits()
    for again in (all_fits(), all_fits()):
        for a, b in zip(first, again):
            assert torch.equal(a, b)
