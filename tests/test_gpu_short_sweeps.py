"""Start and end of a workgroup of the register-resident engines: rows read four features at a time or one by one, sums over the lanes.

The same rows at any stride and alignment give the same bits, and the sums are those of 64 bits to what fp32 kernel values leave (1e-6
of positive terms, see test_gpu_f32_parts.py; 4e-6 for the kernels of the distance, whose exponent is a square root)."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu


def _kernel(X, C, sigma, kind):
    x, c = X.double(), C.double()
    r2 = torch.zeros(X.shape[0], C.shape[0], device=X.device, dtype=torch.float64)
    for k in range(X.shape[1]):
        r2 += (x[:, k, None] - c[None, :, k]) ** 2
    r2 /= float(torch.tensor(sigma, dtype=torch.float32)) ** 2
    return torch.exp(-0.5 * r2) if kind == "gaussian" else torch.exp(-r2.sqrt())


# d around the units of 8 features and the steps of 4; points around half a block of 32, a block, a wavefront's 64 and a workgroup's 256
@pytest.mark.parametrize("kind,cross", [("gaussian", "f16x3"), ("gaussian", "f32"), ("laplacian", "f16x3")])
@pytest.mark.parametrize("n,M,d", [(4097, 1025, 1), (2049, 2047, 4), (1999, 2113, 7), (20000, 1000, 8), (3001, 1504, 12), (5000, 993, 13),
                                   (2561, 1791, 16), (3333, 1313, 28), (2080, 2016, 29), (4001, 1055, 44)])
def test_rows_at_any_alignment(knm, kind, cross, n, M, d):
    ctx = knm.Context()
    ctx.set_kernel(kind)
    ctx.set_cross_term(cross)
    g = torch.Generator(device="cuda").manual_seed(n + d)
    X, C = torch.randn(n, d, generator=g, device="cuda"), torch.randn(M, d, generator=g, device="cuda")
    C[: min(n, M) // 3] = X[: min(n, M) // 3]
    sigma, v = 0.75 * math.sqrt(d), torch.rand(M, 1, generator=g, device="cuda") + 0.1
    K = _kernel(X, C, sigma, kind)
    W = K @ v.double()
    U = K.T @ W
    u, w = knm.knm_prod(X, C, sigma, v, return_w=True, ctx=ctx)
    tol = 1e-6 if kind == "gaussian" else 4e-6
    assert float((w.double() - W).norm() / W.norm()) < tol and float((u.double() - U).norm() / U.norm()) < tol

    def moved(A, pad, off):
        wide = torch.full((A.shape[0] * (A.shape[1] + pad) + off,), 7.0, device="cuda")
        view = wide[off:].reshape(A.shape[0], A.shape[1] + pad)[:, : A.shape[1]]
        view.copy_(A)
        return view

    for pad, off in [(1, 0), (4, 0), (0, 1), (4, 2)]:
        u2, w2 = knm.knm_prod(moved(X, pad, off), moved(C, pad, off), sigma, v, return_w=True, ctx=ctx)
        assert torch.equal(u, u2) and torch.equal(w, w2), (pad, off)
