"""The fp32 cross term from three bf16 parts (large products with up to 14 features in the fp32 mode) against 64 bits.

Error bound of the rows used here: an exponent is a sum of terms of at most 16 in size, rounded to 2^-24 of that when the large terms
come in, so a kernel value is off by at most about 1e-6 of itself; weights are positive, so sums are no further off.
"""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu

TOL = 1e-6


@pytest.fixture
def f32(knm):
    ctx = knm.Context()
    ctx.set_cross_term("f32")
    return ctx


def _rows(n, d, seed):
    return torch.randn(n, d, generator=torch.Generator(device="cuda").manual_seed(seed), device="cuda")


def _kernel(X, C, sigma):
    s = float(torch.tensor(sigma, dtype=torch.float32))
    x, c = X.double(), C.double()
    return torch.exp(-((x * x).sum(1)[:, None] + (c * c).sum(1)[None] - 2.0 * x @ c.T).clamp_(min=0.0) / (2.0 * s * s))


def _reference(X, C, sigma, v, w=None):
    W, U = [], torch.zeros(C.shape[0], 1, device="cuda", dtype=torch.float64)
    for lo in range(0, X.shape[0], 16384):
        K = _kernel(X[lo:lo + 16384], C, sigma)
        W.append(K @ v.double())
        U += K.T @ (W[-1] if w is None else W[-1] * w[lo:lo + 16384, None].double())
    return torch.cat(W), U


def _err(got, ref):
    return float((got.double() - ref).norm() / ref.norm())


# the smallest and largest d of every number of matrix instructions; rows and centres around tiles of 32, stages of 128 and 256 and
# blocks of 256; just above the size from which these sweeps are taken
@pytest.mark.parametrize("n,M,d", [(65537, 2049, 1), (65279, 2111, 4), (40961, 2559, 5), (60001, 1793, 6), (70001, 1537, 7), (50000, 2048, 9),
                                   (131101, 769, 10), (255, 300001, 12), (40001, 1601, 13), (64000, 1001, 14), (49153, 1281, 15),
                                   (1025, 65535, 16)])
def test_parts_against_64_bits(knm, f32, n, M, d):
    X, C = _rows(n, d, d), _rows(M, d, 100 + d)
    C[: min(M, n) // 2] = X[: min(M, n) // 2]  # centres among the rows
    sigma = 0.75 * math.sqrt(d)
    v = _rows(M, 1, 7).abs() + 0.1
    W, U = _reference(X, C, sigma, v)
    got, w = knm.knm_prod(X, C, sigma, v, return_w=True, ctx=f32)
    assert _err(w, W) < TOL and _err(got, U) < TOL
    wgt = _rows(n, 1, 8).abs().flatten()
    _, Uw = _reference(X, C, sigma, v, wgt)
    assert _err(knm.knm_prod_weighted(X, C, sigma, wgt, v, ctx=f32), Uw) < TOL
    # a leading dimension larger than d and rows that start at any multiple of four bytes
    wide = torch.full((n, d + 3), float("nan"), device="cuda")
    wide[:, 1:1 + d] = X
    assert torch.equal(knm.knm_prod(wide[:, 1:1 + d], C, sigma, v, ctx=f32), got)


def test_parts_do_not_depend_on_the_workspace(knm, f32):
    X, C = _rows(300001, 9, 1), _rows(1501, 9, 2)
    v = _rows(1501, 1, 3)
    U = knm.knm_prod(X, C, 2.0, v, ctx=f32)
    Us, Ws = torch.empty_like(U), torch.empty(300001, 1, device="cuda")
    knm.knm_prod_static(X, C, 2.0, v, Ws, Us, ctx=f32)
    assert torch.equal(U, Us)
    f32.set_pack_limit(1 << 20)  # slab by slab
    assert torch.equal(U, knm.knm_prod(X, C, 2.0, v, ctx=f32))


def test_parts_have_no_range_limits(knm, f32):
    """Rows far outside what half precision holds, infinite rows and rows that are not numbers add nothing and leave the others alone."""
    n, M, d = 65537, 2049, 7
    X, C, v = _rows(n, d, 4), _rows(M, d, 5), _rows(M, 1, 6).abs()
    plain = knm.knm_prod(X, C, 2.0, v, return_w=True, ctx=f32)[1]
    far = torch.arange(3, n, 997, device="cuda")
    big = X.clone()
    for i, value in enumerate((1e6, -3e12, 1e25, float("inf"), float("-inf"), float("nan"))):
        big[far[i::6], i] = value
    U, W = knm.knm_prod(big, C, 2.0, v, return_w=True, ctx=f32)
    assert bool((W[far] == 0).all())
    rest = torch.ones(n, dtype=torch.bool, device="cuda")
    rest[far] = False
    assert torch.equal(W[rest], plain[rest])
    assert _err(U, _reference(X[rest], C, 2.0, v)[1]) < TOL


# Bound: U rounded to fp32 is off by 2^-24 / sqrt(3) of itself at most in the rms, about 2.5e-8 over all mantissas; what the matrix cores cut off, always
# to one side, may shift each of the two sums of positive terms by a quarter of its last bit, 3e-8 together.
@pytest.mark.parametrize("d", [1, 2, 3, 4, 6])
def test_what_the_matrix_cores_cut_off_does_not_add_up(knm, f32, d):
    X, v = _rows(40000, d, 30 + d), _rows(9000, 1, 7).abs()
    C, sigma = X[:9000].contiguous(), 0.75 * math.sqrt(d)
    W, U = _reference(X, C, sigma, v)
    assert _err(knm.knm_prod(X, C, sigma, v, ctx=f32), U) < 3.9e-8
