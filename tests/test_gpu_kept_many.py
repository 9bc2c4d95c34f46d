"""Products with many columns whose kernel values are formed once and read for both sums, against 64 bits.

Bound: a kernel value is off by about 4e-7 of itself (22 bits of every feature, fp32 exponent), its two halves and those of the vectors by
2^-22; vectors are positive, so sums are no further off than that and the fp32 sums over a chunk, 1e-6 together.
"""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu

TOL = 2e-6


def _rows(n, d, seed):
    return torch.randn(n, d, generator=torch.Generator(device="cuda").manual_seed(seed), device="cuda")


def _reference(X, C, sigma, V, w=None):
    s = float(torch.tensor(sigma, dtype=torch.float32))
    c, v = C.double(), V.double()
    W, U = [], torch.zeros(C.shape[0], V.shape[1], device="cuda", dtype=torch.float64)
    for lo in range(0, X.shape[0], 8192):
        x = X[lo:lo + 8192].double()
        K = torch.exp(-((x * x).sum(1)[:, None] + (c * c).sum(1)[None] - 2.0 * x @ c.T).clamp_(min=0.0) / (2.0 * s * s))
        W.append(K @ v)
        U += K.T @ (W[-1] if w is None else W[-1] * w[lo:lo + 8192, None].double())
    return torch.cat(W), U


def _err(got, ref):
    return float((got.double() - ref).norm() / ref.norm())


# the smallest d and the edges of the column groups; rows and centres around blocks of 32, tiles of 128 and workgroups of 256; one slab and
# several (the last two); more columns than a launch takes
@pytest.mark.parametrize("n,M,d,t", [(10241, 9985, 450, 13), (30001, 4001, 460, 32), (12289, 8223, 320, 33), (300_000, 353, 325, 64), (511, 200_033, 210, 65),
                                     (20_000, 5120, 211, 128), (16_385, 6337, 180, 129), (40_031, 2559, 181, 160), (10_001, 10_001, 300, 161),
                                     (21_000, 70_001, 180, 144), (20_225, 65_569, 450, 17)])
def test_products_with_many_columns(knm, n, M, d, t):
    X, C = _rows(n, d, 1), _rows(M, d, 2)
    k = min(n, M) // 2
    C[:k] = X[:k]  # centres among the rows
    sigma = 0.75 * math.sqrt(d)
    V = _rows(M, t, 3).abs() + 0.01
    V[:, 1] *= 1e-12  # columns of their own scales
    V[:, 2] *= 1e9
    V[:, t - 1] = 0.0
    W, U = _reference(X, C, sigma, V)
    got, w = knm.knm_prod(X, C, sigma, V, return_w=True)
    assert bool((got[:, t - 1] == 0).all()) and bool((w[:, t - 1] == 0).all())
    for c in range(t - 1):
        assert _err(w[:, c], W[:, c]) < TOL and _err(got[:, c], U[:, c]) < TOL, c
    assert torch.equal(knm.knm_prod(X, C, sigma, V), got)
    wgt = _rows(n, 1, 4).abs().flatten()
    _, Uw = _reference(X, C, sigma, V, wgt)
    weighted = knm.knm_prod_weighted(X, C, sigma, wgt, V)
    for c in range(t - 1):
        assert _err(weighted[:, c], Uw[:, c]) < TOL, c


# Products that would keep their kernel values and cannot: both images beyond the cap, no room for a slab, the call that allocates nothing.  Two sweeps,
# as far from 64 bits as with kept values, and the same to the last bits whatever the reason.
@pytest.mark.parametrize("n,M,d,t", [(20_001, 5001, 320, 33), (30_003, 3400, 460, 17)])
def test_products_with_many_columns_without_kept_values(knm, n, M, d, t):
    X, C = _rows(n, d, 1), _rows(M, d, 2)
    C[:1000] = X[:1000]
    sigma, V = 0.75 * math.sqrt(d), _rows(M, t, 3).abs() + 0.01
    W, U = _reference(X, C, sigma, V)
    kept = knm.knm_prod(X, C, sigma, V, return_w=True)
    ctx = knm.Context()
    ctx.set_pack_limit(1 << 20)
    capped = knm.knm_prod(X, C, sigma, V, return_w=True, ctx=ctx)
    Us, Ws = torch.empty_like(U, dtype=torch.float32), torch.empty_like(W, dtype=torch.float32)
    knm.knm_prod_static(X, C, sigma, V, Ws, Us, ctx=ctx)
    free, total = torch.cuda.mem_get_info()
    others = torch.empty(max(free - total // 16 + (256 << 20), 1), device="cuda", dtype=torch.uint8)
    full = knm.knm_prod(X, C, sigma, V, return_w=True, ctx=knm.Context())
    del others
    torch.cuda.empty_cache()
    for u, w in (kept, capped, full, (Us, Ws)):
        assert _err(w, W) < TOL and _err(u, U) < TOL
    assert torch.equal(capped[0], full[0]) and torch.equal(capped[1], full[1])
    assert not torch.equal(kept[0], full[0])  # (by kept values)
