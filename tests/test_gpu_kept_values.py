"""Products and fits that form kernel values once and read them again, against the oracle."""
import contextlib
import math

import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


def rel_l2(got, ref):
    got, ref = np.asarray(got, dtype=np.float64), np.asarray(ref, dtype=np.float64)
    return float(np.linalg.norm(got - ref) / np.linalg.norm(ref))


def _rand(n, d, seed):
    return torch.randn(n, d, generator=torch.Generator().manual_seed(seed)).to(torch.float32)


# products: the sums over kept rows are those of knm_t_y's sweep to the last bit.  Edges of the 32 x 32 blocks, fixed blocks (256) and tiles
# (128), of 64 centres and of the columns (12), one row, one centre; chunks that end in a slab
@pytest.mark.parametrize("n,M,d,t", [(1, 1, 700, 1), (33, 127, 700, 2), (255, 257, 300, 12), (256, 128, 401, 7), (1000, 511, 784, 10), (2049, 31, 305, 9),
                                     (1537, 1025, 784, 1), (40001, 300, 320, 3), (255, 257, 330, 12)])
def test_products_from_kept_values(knm, n, M, d, t):
    X = _rand(n, d, n + d).cuda()
    C = torch.cat([X[: max(1, M // 2)], _rand(M, d, M).cuda()])[:M].contiguous()  # coincident pairs
    V, w = _rand(M, t, t).cuda(), torch.rand(n, generator=torch.Generator().manual_seed(3)).cuda()
    sigma, ctx = 0.75 * math.sqrt(d), knm.Context()
    U, W = knm.knm_prod(X, C, sigma, V, return_w=True, ctx=ctx)
    assert torch.equal(U, knm.knm_t_y(X, C, sigma, W, ctx=ctx))
    assert torch.equal(knm.knm_prod_weighted(X, C, sigma, w, V, ctx=ctx), knm.knm_t_y(X, C, sigma, W * w[:, None], ctx=ctx))
    some = np.arange(0, n, max(1, n // 500))
    ref = oracle.knm_v(X.cpu().numpy()[some], C.cpu().numpy(), sigma, V.cpu().numpy())
    error = rel_l2(W.cpu().numpy()[some], ref)
    # (W is summed slab by slab; its values carry the same 3e-7 as those of knm_v)
    assert error < 1e-6 and error < 1.5 * rel_l2(knm.knm_v(X, C, sigma, V, ctx=ctx).cpu().numpy()[some], ref) + 1e-7


# two slabs of rows, the second one ragged, with chunks across the boundary; and the announced workspace
@pytest.mark.parametrize("t", [1, 10])
def test_product_in_slabs(knm, t):
    n, M, d = 55003, 25000, 400
    g = torch.Generator(device="cuda").manual_seed(1)
    X = torch.randn(n, d, generator=g, device="cuda")
    C, V, ctx = X[:M].contiguous(), torch.randn(M, t, generator=g, device="cuda"), knm.Context()
    U, W = knm.knm_prod(X, C, 16.0, V, return_w=True, ctx=ctx)
    assert 1 << 31 < ctx.workspace_held() <= knm.load_library().knm_workspace_bytes(n, M, d, t)
    assert torch.equal(U, knm.knm_t_y(X, C, 16.0, W, ctx=ctx))
    v = knm.knm_v(X, C, 16.0, V, ctx=ctx)
    assert float((W - v).norm() / v.norm()) < 1e-6


# a captured product that keeps a slab: fits and larger workspaces in between do not take it away, and every replay is the eager result
def test_product_with_a_slab_replays_in_a_graph(knm):
    n, M, d, t, sigma = 3000, 700, 784, 10, 21.0
    X, C, V, w = _rand(n, d, 70).cuda(), _rand(M, d, 71).cuda(), _rand(M, t, 72).cuda(), torch.rand(n, generator=torch.Generator().manual_seed(4)).cuda()
    U, Z, Y = torch.empty(M, t, device="cuda"), torch.empty(M, t, device="cuda"), _rand(4000, 2, 73).cuda()
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        ctx = knm.Context()  # bound to the side stream
        for graph in (None, torch.cuda.CUDAGraph()):  # an eager call allocates the workspace
            with contextlib.ExitStack() as stack:
                if graph is not None:
                    stack.enter_context(torch.cuda.graph(graph, stream=side))
                knm.knm_prod(X, C, sigma, V, out=U, ctx=ctx)
                Z.copy_(knm.knm_prod_weighted(X, C, sigma, w, V, ctx=ctx))
            side.synchronize()
    F = _rand(4000, 300, 74).cuda()
    for rep in range(4):
        print(f"replay {rep}", flush=True)
        X.copy_(_rand(n, d, 80 + rep).cuda())
        V.copy_(_rand(M, t, 90 + rep).cuda())
        U.fill_(float("nan"))
        Z.fill_(float("nan"))
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            knm.falkon_fit(F, Y, F[: 100 * (rep + 1)], 13.0, 1e-4, 3, 1e-6, ctx=ctx)
            graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(U, knm.knm_prod(X, C, sigma, V)) and torch.equal(Z, knm.knm_prod_weighted(X, C, sigma, w, V)), rep
    del graph
    ctx.close()


# slabs with fewer rows than there are centres, the first of them far from everything else: the common shift is the whole pair's (that of the
# first slab left an error of 4e-3 in W and another U than knm_t_y's)
def test_product_in_slabs_of_sorted_rows(knm):
    n, M, d, sigma = 40000, 36000, 400, 16.0
    g = torch.Generator(device="cuda").manual_seed(2)
    X = torch.randn(n, d, generator=g, device="cuda")
    X[:16384] += 100.0 * sigma / math.sqrt(d)
    C, V, ctx = torch.randn(M, d, generator=g, device="cuda"), torch.randn(M, 2, generator=g, device="cuda"), knm.Context()
    C[::2] = X[-18000:]
    U, W = knm.knm_prod(X, C, sigma, V, return_w=True, ctx=ctx)
    assert ctx.workspace_held() > 16384 * M * 4  # a slab of values
    assert torch.equal(U, knm.knm_t_y(X, C, sigma, W, ctx=ctx))
    some = np.r_[0:16384:128, 16384:n:128]
    ref, other = (oracle.knm_v(X[some].cpu().numpy(), C.cpu().numpy(), sigma, v.cpu().numpy()) for v in (V, V.abs()))
    assert rel_l2(W[some].cpu().numpy(), ref) < 1e-6
    assert np.abs(W[some].cpu().numpy() - ref).max() < 1e-6 * other.max()


# fits: one and two groups of columns, kernels of r (every centre coincides with a row), the fp32 engine; sizes at the edges of the 32 x 32 blocks,
# the fixed blocks (256) and the tiles (128), one of them the smallest there is.  Predictions carry what the products' rounding (3e-7)
# becomes through T^-1 at this jitter, and no more than those of sweeps that form the values each time (1e-5)
@pytest.mark.parametrize("n,M,d,t,cross,kernel", [(1100, 130, 400, 1, "f16x3", "gaussian"), (900, 257, 784, 20, "f16x3", "gaussian"),
                                                  (256, 128, 700, 16, "f16x3", "gaussian"), (1537, 33, 705, 17, "f16x3", "gaussian"),
                                                  (1, 1, 700, 1, "f16x3", "gaussian"), (700, 100, 300, 3, "f16x3", "laplacian"),
                                                  (513, 255, 301, 9, "f16x3", "matern52"), (1025, 128, 90, 2, "f32", "gaussian"),
                                                  (257, 31, 91, 32, "f32", "laplacian")])
def test_fits_from_kept_values(knm, n, M, d, t, cross, kernel):
    X, Y, Xt, sigma = _rand(n, d, n), _rand(n, t, t), _rand(200, d, 8), 0.5 * math.sqrt(d)
    C = X[:M].clone()
    ctx = knm.Context()
    ctx.set_cross_term(cross)
    ctx.set_kernel(kernel)
    alpha = knm.falkon_fit(X.cuda(), Y.cuda(), C.cuda(), sigma, 1e-4, 8, 1e-6, ctx=ctx)
    assert torch.equal(alpha, knm.falkon_fit(X.cuda(), Y.cuda(), C.cuda(), sigma, 1e-4, 8, 1e-6, ctx=ctx))
    got = knm.falkon_predict(Xt.cuda(), C.cuda(), sigma, alpha, ctx=ctx).cpu().numpy()
    with oracle.kernel(kernel):
        ao = oracle.falkon_fit(X.numpy(), Y.numpy(), C.numpy(), sigma, 1e-4, 8, 1e-6)
        ref = oracle.falkon_predict(Xt.numpy(), C.numpy(), sigma, ao)
    print(rel_l2(got, ref))
    assert rel_l2(got, ref) < 1e-4


# the logistic fit: weighted sums over kept values, and k(C, C) beside them; also X as its own centres
@pytest.mark.parametrize("n,M", [(1500, 300), (400, 400)])
def test_logistic_fit_from_kept_values(knm, n, M):
    d = 500
    X, sigma = _rand(n, d, n), 0.5 * math.sqrt(d)
    y = torch.where(X[:, :1] + 0.5 * X[:, 1:2] * X[:, 2:3] > 0, 1.0, -1.0)
    C, yC = (X, y) if M == n else (X[:M].clone(), y[:M].clone())
    Xd = X.cuda()
    Cd = Xd if M == n else C.cuda()
    alpha, loss = knm.logfalkon_fit(Xd, y.cuda(), Cd, yC.cuda(), sigma, [1e-2, 1e-3], [4, 5], 1e-6, return_loss=True)
    ao, lo = oracle.logfalkon_fit(X.numpy(), y.numpy(), C.numpy(), yC.numpy(), sigma, [1e-2, 1e-3], [4, 5], 1e-6, return_loss=True)
    Xt = _rand(200, d, 9)
    pred = knm.falkon_predict(Xt.cuda(), Cd, sigma, alpha).cpu().numpy()
    assert rel_l2(pred, oracle.falkon_predict(Xt.numpy(), C.numpy(), sigma, ao)) < 1e-3
    assert np.allclose(loss, lo, rtol=1e-4, atol=1e-6)


# centres that are views of the rows, or rows that are a view of the centres: the result of copies of them, to the last bit, from kept values
@pytest.mark.parametrize("cross", ["f16x3", "f32"])
@pytest.mark.parametrize("which", ["every tenth row", "first rows", "rows among the centres"])
def test_logistic_fit_of_views_from_kept_values(knm, which, cross):
    d, sigma = 500, 0.5 * math.sqrt(500)
    P = _rand(3000, d, 21)
    z = torch.where(P[:, :1] + 0.5 * P[:, 1:2] * P[:, 2:3] > 0, 1.0, -1.0).cuda()
    P = P.cuda()
    X, y, C, yC = {"every tenth row": (P, z, P[::10], z[::10].contiguous()), "first rows": (P, z, P[:300], z[:300]),
                   "rows among the centres": (P[:300], z[:300], P[:1000], z[:1000])}[which]
    fits = []
    for copied in (True, False):
        ctx = knm.Context()
        ctx.set_cross_term(cross)
        fits.append(knm.logfalkon_fit(X.clone() if copied else X, y, C.clone() if copied else C, yC, sigma, [1e-2, 1e-3], [4, 5], 1e-6, ctx=ctx))
    assert torch.equal(*fits)
    ao = oracle.logfalkon_fit(X.cpu().numpy(), y.cpu().numpy(), C.cpu().numpy(), yC.cpu().numpy(), sigma, [1e-2, 1e-3], [4, 5], 1e-6)
    Xt = _rand(200, d, 9)
    pred = knm.falkon_predict(Xt.cuda(), C, sigma, fits[0]).cpu().numpy()
    assert rel_l2(pred, oracle.falkon_predict(Xt.numpy(), C.cpu().numpy(), sigma, ao)) < 1e-3
