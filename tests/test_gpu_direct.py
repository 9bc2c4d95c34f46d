"""Small predictions in one launch, against the oracle: edges of the rows and centres of a workgroup, split rows, all kernels."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


def _rand(n, d, seed):
    return torch.randn(n, d, generator=torch.Generator().manual_seed(seed)).to(torch.float32)


# rows per workgroup 4, 2, 1 by the columns; one centre, fewer and more than a workgroup's 256, rows split over workgroups
@pytest.mark.parametrize("kernel", ["gaussian", "laplacian", "matern32", "matern52"])
@pytest.mark.parametrize("n,M,d,t", [(1, 1, 1, 1), (5, 255, 3, 2), (4, 257, 8, 3), (203, 1000, 9, 4), (3, 4097, 128, 7), (1, 50001, 5, 1), (17, 2049, 100, 16),
                                     (1000, 300, 12, 1), (2, 9000, 44, 9)])
def test_small_predictions(knm, kernel, n, M, d, t):
    C = _rand(M, d, M)
    X = torch.cat([C[: min(M, (n + 1) // 2)], _rand(n, d, n)])[:n].contiguous()  # coincident pairs
    V, sigma = _rand(M, t, t), float(np.float32(0.75 * d ** 0.5))
    ctx = knm.Context()
    ctx.set_kernel(kernel)
    got = knm.falkon_predict(X.cuda(), C.cuda(), sigma, V.cuda(), ctx=ctx).cpu().numpy().astype(np.float64)
    with oracle.kernel(kernel):
        ref = oracle.knm_v(X.numpy(), C.numpy(), sigma, V.numpy())
        scale = oracle.knm_v(X.numpy(), C.numpy(), sigma, np.abs(V.numpy()))
    # d differences, squares and sums of 2^-24 each in the exponent (at most 15 or so where the value counts), the exponential, 16 terms
    # and 8 levels of fp32 sums: below 2e-6 of the sum of magnitudes, and a tenth of that in the 2-norm
    assert np.max(np.abs(got - ref) / scale) < 2e-6
    assert np.linalg.norm(got - ref) < 5e-7 * np.linalg.norm(scale)


# any leading dimension and alignment gives the same result
def test_small_predictions_of_views(knm):
    big, C, V = _rand(60, 40, 1).cuda(), _rand(600, 41, 2).cuda(), _rand(600, 1, 3).cuda()
    X = big[:50, 3:19]
    for Cv in (C[:500, :16], C[:500, 1:17], C[7:507, 4:20]):
        a = knm.knm_v(X, Cv, 3.0, V[:500])
        b = knm.knm_v(X.contiguous(), Cv.contiguous(), 3.0, V[:500].contiguous())
        assert torch.equal(a, b)


# nothing is clamped, but points beyond the range of the split-fp16 mode are reported in it, wherever the data lies
@pytest.mark.parametrize("where,index", [("X", 0), ("X", 77), ("C", 0), ("C", 290)])
def test_small_predictions_report_the_range(knm, where, index):
    X, C, V, ctx = _rand(100, 6, 1) + 5.0e3, _rand(300, 6, 2) + 5.0e3, _rand(300, 1, 3), knm.Context()
    knm.knm_v(X.cuda(), C.cuda(), 1.0, V.cuda(), ctx=ctx)
    assert ctx.range_exceeded() == 0
    (X if where == "X" else C)[index, 5] += 3.0e3
    W = knm.knm_v(X.cuda(), C.cuda(), 1.0, V.cuda(), ctx=ctx).cpu().numpy()
    assert ctx.range_exceeded() >= 1
    ref, scale = (oracle.knm_v(X.numpy(), C.numpy(), 1.0, v) for v in (V.numpy(), np.abs(V.numpy())))
    assert np.linalg.norm(W - ref) < 2e-6 * np.linalg.norm(scale)
    ctx.set_cross_term("f32")
    knm.knm_v(X.cuda(), C.cuda(), 1.0, V.cuda(), ctx=ctx)
    assert ctx.range_exceeded() == 0


# what is reported is what the engines report (knm_prod's row sweep packs the same points): outliers in the first row, the first centre, both or
# neither, on either side of 1705 sigma from the smaller set's mean; sets far from the origin, from each other and spread
# out; points in range but more than that apart.  Nothing lies within a tenth of the line
@pytest.mark.parametrize("n,M", [(100, 300), (300, 100), (40, 4200), (1, 600), (1, 1)])
@pytest.mark.parametrize("name", ["opposite outliers in range", "first points out together", "one beyond", "one far row", "sets far from the origin",
                                  "sets apart", "sets a little apart", "spread out", "spread beyond", "rows beyond beside the first centre",
                                  "centres beyond beside the first rows", "a NaN"])
def test_small_predictions_report_what_the_engines_would(knm, n, M, name):
    if name == "a NaN" and M == 1:
        pytest.skip("the engines' shift is that of the row")
    d, ctx = 6, knm.Context()
    X, C, V = _rand(n, d, n), _rand(M, d, M + 1), _rand(M, 1, 3)
    if name == "opposite outliers in range":
        X[n // 2, 1] += 1500.0
        C[0, 1] -= 1500.0 if n > 1 else 0.0
    elif name == "first points out together":
        X[0] += 1000.0
        C[0] += 1000.0
    elif name == "one beyond":
        C[M // 3, 2] += 1900.0 if M > 1 else 0.0
    elif name == "one far row":
        X[n - 1, 2] += 1500.0
    elif name == "sets far from the origin":
        X += 1.0e5
        C += 1.0e5
    elif name == "sets apart":
        X[:, 0] += 2000.0
    elif name == "sets a little apart":
        X[:, 0] += 1200.0
        C[:, 0] -= 200.0
    elif name == "spread out":
        X[:, 0] = torch.linspace(-1400.0, 1400.0, n) if n > 1 else X[:, 0]
        C[:, 0] = torch.linspace(1400.0, -1400.0, M) if M > 1 and n > 1 else C[:, 0]
    elif name == "spread beyond":
        X[:, 0] = torch.linspace(-2100.0, 2100.0, n)
        C[:, 0] = torch.linspace(2100.0, -2100.0, M)
    elif name == "rows beyond beside the first centre":  # which is in range, and less than a third of it away
        X[-4:, 1] += 2090.0
        C[0, 1] += 1535.0
    elif name == "centres beyond beside the first rows":  # all of a workgroup's, where there are 4200
        X[:4, 1] += 1535.0
        C[-104:, 1] += 2090.0
    else:
        X[n // 2, 3] = float("nan")
    X, C, V = X.cuda(), C.cuda(), V.cuda()
    knm.knm_prod(X, C, 1.0, V, ctx=ctx)
    engines = ctx.range_exceeded()
    knm.knm_v(X, C, 1.0, V, ctx=ctx)
    small = ctx.range_exceeded()
    print(name, engines, small)
    assert (small > 0) == (engines > 0)


# units in which squares leave fp32: sigma and the features times a power of two give the same result
@pytest.mark.parametrize("power", [-80, -66, -50, 50, 66, 80])
def test_small_predictions_in_any_unit(knm, power):
    X, C, V, unit = _rand(100, 8, 1).cuda(), _rand(300, 8, 2).cuda(), _rand(300, 2, 3).cuda(), 2.0 ** power
    W = knm.knm_v(X, C, 2.0, V)
    other = knm.knm_v(X * unit, C * unit, 2.0 * unit, V)
    assert float((other - W).norm() / W.norm()) < 2e-6


# a point that is not finite, or too far for its square to be, has the value 0 in the split-fp16 mode and for the Gaussian kernel: its row is 0, and the other
# rows are what they are without it.  Kernels of r in the fp32 mode carry a NaN on
@pytest.mark.parametrize("cross", ["f16x3", "f32"])
@pytest.mark.parametrize("kernel", ["gaussian", "laplacian", "matern32", "matern52"])
@pytest.mark.parametrize("n,M,d,t", [(100, 300, 6, 1), (100, 300, 8, 3), (5, 4200, 8, 1)])
@pytest.mark.parametrize("value", [float("nan"), float("inf"), -float("inf"), 1e25, 1e18])
def test_small_predictions_with_a_point_that_is_not_finite(knm, n, M, d, t, value, kernel, cross):
    ctx = knm.Context()
    ctx.set_kernel(kernel)
    ctx.set_cross_term(cross)
    X, C, V, sigma = _rand(n, d, 1), _rand(M, d, 2), _rand(M, t, 3), 1.5
    far_row, far_centre, without = X.clone(), C.clone(), V.clone()
    far_row[n // 2, 2] = far_centre[M // 3, 2] = value
    without[M // 3] = 0.0
    row, centre, both = (knm.knm_v(x.cuda(), c.cuda(), sigma, V.cuda(), ctx=ctx).cpu().numpy().astype(np.float64)
                         for x, c in ((far_row, C), (X, far_centre), (far_row, far_centre)))
    with oracle.kernel(kernel):
        ref, other, scale = (oracle.knm_v(X.numpy(), C.numpy(), sigma, v.numpy()) for v in (V, without, V.abs()))
    rest = np.arange(n) != n // 2
    if cross == "f32" and kernel != "gaussian" and not abs(value) < 1e20:
        if value != value:
            assert np.isnan(row[n // 2]).all() and np.isnan(centre).all()
        assert np.max(np.abs(row - ref)[rest] / scale[rest]) < 2e-6
        return
    assert (row[n // 2] == 0.0).all() and np.max(np.abs(row - ref)[rest] / scale[rest]) < 2e-6
    assert np.max(np.abs(centre - other) / scale) < 2e-6
    if value != value:
        assert (both[n // 2] == 0.0).all() and np.max(np.abs(both - other)[rest] / scale[rest]) < 2e-6
