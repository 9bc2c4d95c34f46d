"""Packed images and shift that several sweeps share: the forms in which the sets of a sweep are not simply (X, C) and (C, X)."""
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


# X is C: one image serves as fixed and as stream operand (vector-ALU reduction, matrix-core reduction, register-resident engine);
# sizes with whole and ragged fixed blocks and chunks
@pytest.mark.parametrize("d,t", [(200, 10), (60, 1), (60, 20), (30, 144), (28, 1)])
@pytest.mark.parametrize("n", [512, 2049, 3000])
def test_products_of_a_set_with_itself(knm, n, d, t):
    X, V, sigma = _rand(n, d, n + d), _rand(n, t, t), 0.75 * d ** 0.5
    Xd, Vd = X.cuda(), V.cuda()
    U, W = knm.knm_prod(Xd, Xd, sigma, Vd, return_w=True)
    U2, W2 = knm.knm_prod(Xd, Xd.clone(), sigma, Vd, return_w=True)
    assert torch.equal(U, U2) and torch.equal(W, W2)
    rows = np.arange(0, n, 37)
    assert rel_l2(W.cpu().numpy()[rows], oracle.knm_v(X.numpy()[rows], X.numpy(), sigma, V.numpy())) < 1e-5


# a fit on its own centres: every sweep is k(X, X)
def test_fit_of_a_set_on_itself(knm):
    n, d, t = 1500, 60, 10
    X, Y, sigma = _rand(n, d, 3).cuda(), _rand(n, t, 4).cuda(), 6.0
    a = knm.falkon_fit(X, Y, X, sigma, 1e-4, 6, 1e-6)
    b = knm.falkon_fit(X, Y, X.clone(), sigma, 1e-4, 6, 1e-6)
    assert torch.equal(a, b)


# the first sweep of a fit clamps operands when images are already kept: the rest runs as if the fp32 mode had been set
@pytest.mark.parametrize("d,t", [(60, 3), (200, 1), (28, 1)])
def test_fallback_with_kept_images(knm, d, t):
    n, M, sigma = 5000, 300, 0.75 * d ** 0.5
    X, Y = _rand(n, d, 5), _rand(n, t, 6)
    C = X[:M].clone()
    X[M + 7, 2] = 5.0e5
    ctx = knm.Context()
    got = knm.falkon_fit(X.cuda(), Y.cuda(), C.cuda(), sigma, 1e-5, 5, 1e-7, ctx=ctx)
    assert ctx.range_exceeded() >= 1 and ctx.cross_term == "f16x3"
    ctx32 = knm.Context()
    ctx32.set_cross_term("f32")
    assert torch.equal(got, knm.falkon_fit(X.cuda(), Y.cuda(), C.cuda(), sigma, 1e-5, 5, 1e-7, ctx=ctx32))
    # and the context's next fit, on ordinary data, keeps split-fp16 images again
    X[M + 7, 2] = 0.0
    again = knm.falkon_fit(X.cuda(), Y.cuda(), C.cuda(), sigma, 1e-5, 5, 1e-7, ctx=ctx)
    assert torch.equal(again, knm.falkon_fit(X.cuda(), Y.cuda(), C.cuda(), sigma, 1e-5, 5, 1e-7, ctx=knm.Context()))
    assert ctx.range_exceeded() == 0


# logistic fits on the K-loop engine: the sweep k(C, C) of every Newton step shares shift and images with those over X, for centres of
# fewer and of more than a fixed block, and X as its own centres
@pytest.mark.parametrize("n,M,d", [(4000, 250, 60), (3000, 700, 120), (600, 600, 60)])
def test_logistic_fit_on_the_k_loop_engine(knm, n, M, d):
    X, sigma, jitter = _rand(n, d, n), 0.75 * d ** 0.5, 1e-6
    y = torch.where(X[:, :1] + 0.5 * X[:, 1:2] * X[:, 2:3] > 0, 1.0, -1.0)
    C, yC = (X, y) if M == n else (X[:M].clone(), y[:M].clone())
    Xd = X.cuda()
    Cd = Xd if M == n else C.cuda()
    lambdas, iters = [1e-2, 1e-3, 1e-4], [4, 4, 6]
    alpha, loss = knm.logfalkon_fit(Xd, y.cuda(), Cd, yC.cuda(), sigma, lambdas, iters, jitter, return_loss=True)
    ao, lo = oracle.logfalkon_fit(X.numpy(), y.numpy(), C.numpy(), yC.numpy(), sigma, lambdas, iters, jitter, return_loss=True)
    Xt = _rand(500, d, 9)
    pred = knm.falkon_predict(Xt.cuda(), Cd, sigma, alpha).cpu().numpy()
    assert rel_l2(pred, oracle.falkon_predict(Xt.numpy(), C.numpy(), sigma, ao)) < 1e-3
    assert np.allclose(loss, lo, rtol=1e-4, atol=1e-6)
