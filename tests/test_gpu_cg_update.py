"""The vector steps of an iteration of CG, in one launch up to M = 4096: fits against the same iterations in 64 bits on formed kernel blocks.

With jitter and lambda of 1e-2 the inverses of the two factors are at most 10 in norm and each is applied twice between a product and the
coefficients: the rounding of the products, 3e-7, grows by at most 1e4."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu


def _kernel(a, b, sigma):
    a, b = a.double(), b.double()
    return torch.exp(-((a * a).sum(1)[:, None] + (b * b).sum(1)[None] - 2.0 * a @ b.T).clamp_(min=0.0) / (2.0 * sigma * sigma))


# around a wavefront, a workgroup of the partial sums, the next number of those and the largest M of one launch
@pytest.mark.parametrize("t", [1, 3])
@pytest.mark.parametrize("M", [1, 63, 256, 257, 1023, 1024, 1025, 2049, 3073, 4095, 4096, 4097])
def test_iterations_against_64_bits(knm, M, t):
    n, d, lam, jitter, iters = 6000, 10, 1e-2, 1e-2, 6
    g = torch.Generator(device="cuda").manual_seed(M + t)
    X = torch.randn(n, d, generator=g, device="cuda")
    C, Y = X[:M].contiguous(), torch.randn(n, t, generator=g, device="cuda") + X[:, :1]
    sigma = float(torch.tensor(0.75 * math.sqrt(d), dtype=torch.float32))
    got = knm.falkon_fit(X, Y, C, sigma, lam, iters, jitter).double()

    K, eye = _kernel(X, C, sigma), torch.eye(M, device="cuda", dtype=torch.float64)
    T = torch.linalg.cholesky(_kernel(C, C, sigma) + jitter * eye).T
    A = torch.linalg.cholesky(T @ T.T / M + lam * eye).T
    solve = torch.linalg.solve_triangular

    def back(u):
        return solve(A.T, u, upper=False)

    def apply(p):
        v = solve(A, p, upper=True)
        z = solve(T, v, upper=True)
        return back(solve(T.T, K.T @ (K @ z), upper=False) + lam * n * v)

    r = back(solve(T.T, K.T @ Y.double(), upper=False))
    b, p, rho = torch.zeros_like(r), r.clone(), (r * r).sum(0)
    for _ in range(iters):
        q = apply(p)
        a = torch.nan_to_num(rho / (p * q).sum(0))  # (0 / 0 once M = 1 has converged)
        b, r = b + a * p, r - a * q
        rho, old = (r * r).sum(0), rho
        p = r + torch.nan_to_num(rho / old) * p
    want = solve(T, solve(A, b, upper=True), upper=True)
    assert float((got - want).norm() / want.norm()) < 3e-3
