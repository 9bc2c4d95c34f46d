"""The preconditioner's symmetric updates as integer products modulo small numbers (block rows and triangular products from a few
thousand centres on): the identities that the factors satisfy, and bit-for-bit repetition.

Bound: an entry of the identities is a sum of some tens of updates, each rounded once in C (2^-53 of it) and off by at most 2^-57 of
the two rows' norms in the operands: below 2e-15 with rows of norm about 1.  The products that check them are running sums of
M terms that stay below 1, rounded to 2^-53 every time: sqrt(M) of that, and the largest of all entries up to four times as much.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _bound(M):
    return 4.0 * 2.0 ** -53 * M ** 0.5


def _centres(M, d, seed):
    return torch.randn(M, d, generator=torch.Generator(device="cuda").manual_seed(seed), device="cuda")


def _factors(pre):
    T, A = pre.factors()
    return torch.from_numpy(T).cuda(), torch.from_numpy(A).cuda()


def _kmm(C, sigma, jitter):
    s = float(torch.tensor(sigma, dtype=torch.float32))
    q = torch.zeros(C.shape[0], C.shape[0], device="cuda", dtype=torch.float64)
    for x in C.double().T:
        q += (x[:, None] - x[None]) ** 2
    K = torch.exp(-q / (2.0 * s * s))
    K.diagonal().add_(jitter)
    return K


# triangular products alone (from 3488 centres on), block rows as well (from 5304 on); tiles of 256 x 128 with remainders, several slabs of the
# contraction
@pytest.mark.parametrize("M", [3600, 4609, 6145, 8191, 13057])
def test_factors_from_residues(knm, M):
    d, sigma, lam, jitter = 5, 1.2, 1e-6, 1e-5
    C = _centres(M, d, M)
    pre = knm.precond_build(C, sigma, lam, jitter)
    T, A = _factors(pre)
    eye = torch.eye(M, device="cuda", dtype=torch.float64)
    assert float((T.T @ T - _kmm(C, sigma, jitter)).abs().max()) < _bound(M)
    B = T @ T.T / M + lam * eye
    assert float((A.T @ A - B).abs().max()) < _bound(M) * float(B.diagonal().max())
    again = knm.precond_build(C, sigma, lam, jitter)
    T2, A2 = _factors(again)
    assert torch.equal(T, T2) and torch.equal(A, A2)
    again.close()
    pre.close()


@pytest.mark.parametrize("M,weights", [(3700, "positive"), (4700, "signed"), (4500, "zeros"), (4500, "wide"), (6145, "signed")])
def test_weighted_products_from_residues(knm, M, weights):
    d, sigma, jitter = 6, 1.4, 1e-5
    C = _centres(M, d, 1)
    g = torch.Generator(device="cuda").manual_seed(2)
    w = torch.rand(M, generator=g, device="cuda", dtype=torch.float64) * 0.25
    lam = 1e-5
    if weights == "signed":
        w[::7] *= -1e-3  # (the identity holds for weights of either sign)
        lam = 1.0
    elif weights == "zeros":
        w[::3] = 0.0
    elif weights == "wide":
        w *= 10.0 ** (-12.0 * torch.rand(M, generator=g, device="cuda", dtype=torch.float64))
    pre = knm.precond_build(C, sigma, 1.0, jitter)
    pre.reweight(lam, w)
    T, A = _factors(pre)
    B = (T * w) @ T.T / M + lam * torch.eye(M, device="cuda", dtype=torch.float64)
    scale = B.diagonal().sqrt()
    assert float(((A.T @ A - B).abs() / (scale[:, None] * scale[None])).max()) < _bound(M)
    pre.close()


def test_weights_that_are_not_numbers_are_reported(knm):
    M = 4500
    pre = knm.precond_build(_centres(M, 6, 3), 1.4, 1.0, 1e-5)
    for value in (float("nan"), float("inf")):
        w = torch.full((M,), 0.1, device="cuda", dtype=torch.float64)
        w[M // 2] = value
        with pytest.raises(knm.KnmError) as e:
            pre.reweight(1e-5, w)
        assert e.value.status == -5
    pre.close()
    C = _centres(5000, 6, 4)
    C[1000:2000] = C[0]  # equal centres without a jitter: not positive definite
    with pytest.raises(knm.KnmError) as e:
        knm.precond_build(C, 1.4, 1e-5, 0.0)
    assert e.value.status == -5


# ---- the update itself, against sums in extended precision ----
#
# Rows of norm about 1 with one large entry at a place of their own, all others about 2^-20: the sum of two rows is a large entry of each times a small one of
# the other, 2^-20, whose rounding is no matter, so that what is left is the rounding of the operands.  Scaled to norms in (2^57, 2^58], entries are rounded by
# at most half a unit, 2^-58 of the norm, two of which meet large entries; the others add 2^-20 sqrt(K) of that.
def _spiked_rows(n, K, triangular, weights, seed):
    g = np.random.default_rng(seed)
    a = g.standard_normal((n, K)) * 2.0 ** -20
    a[np.arange(n), np.arange(n) % K] = g.uniform(1.0, 2.0, n) * g.choice([-1.0, 1.0], n)
    a *= 10.0 ** g.uniform(-30, 30, (n, 1))  # rows of their own magnitude
    if triangular:
        a = np.triu(a)
    w = None
    if weights is not None:
        w = g.uniform(0.5, 2.0, K)
        if weights == "signed":
            w[g.random(K) < 0.4] *= -1.0
    return a, w


@pytest.mark.parametrize("n,K,form_nt,lower,slab,triangular,weights", [
    (1, 1, 0, 0, 0, 0, None), (33, 63, 0, 0, 0, 0, None), (127, 64, 1, 0, 0, 0, None), (128, 65, 1, 1, 0, 0, None), (257, 130, 0, 1, 0, 0, None),
    (385, 191, 0, 0, 64, 0, None), (300, 129, 1, 0, 64, 0, "positive"), (255, 200, 1, 1, 128, 0, "signed"), (513, 513, 1, 1, 0, 1, None),
    (511, 511, 1, 0, 192, 1, "positive"), (641, 641, 1, 1, 128, 1, "signed"), (400, 400, 1, 1, 64, 1, "signed")])
def test_update_by_residues(knm, n, K, form_nt, lower, slab, triangular, weights):
    a, w = _spiked_rows(n, K, triangular, weights, n + K)
    wide = a.astype(np.longdouble)
    want = (wide * w if w is not None else wide) @ wide.T
    norm = np.sqrt(((wide * wide) * (np.abs(w) if w is not None else 1.0)).sum(1)).astype(np.float64)
    stored = np.where(np.tril(np.ones((n, K), bool), -1), np.nan, a) if triangular else a  # (below the diagonal anything may be)
    A = torch.from_numpy(np.ascontiguousarray(stored.T if form_nt else stored)).cuda()
    alpha, beta, shift = 0.75, -2.0, 3.0
    old = np.random.default_rng(7).standard_normal((n, n)) * np.outer(norm, norm) * 2.0 ** -30
    kept = np.triu(np.ones((n, n), bool))  # entries (i, j), i <= j
    C = torch.from_numpy(np.ascontiguousarray(np.where(kept, old, np.nan) if lower else np.where(kept, old, np.nan).T)).cuda()
    ctx, lib = knm.default_context(), knm.load_library()
    W = None if w is None else torch.from_numpy(w).cuda()
    ctx.check(lib.precond_residue_update(ctx._h, form_nt, lower, n, K, slab, alpha, A.data_ptr(), A.shape[1], None if W is None else W.data_ptr(),
                                         triangular, beta, shift, C.data_ptr(), n))
    got = C.cpu().numpy() if lower else C.cpu().numpy().T
    assert np.isnan(got[~kept]).all()  # the other triangle is neither read nor written
    want = np.longdouble(alpha) * want + np.longdouble(beta) * old + np.longdouble(shift) * np.eye(n)
    # the sum is rounded three times on its way from the integer, the result twice more; a weight's roots and their products with the rows four times
    size = alpha * (np.abs(wide) * (np.abs(w) if w is not None else 1.0)) @ np.abs(wide.T) + 2.0 * np.abs(old) + 3.0 * np.eye(n)
    error = np.abs(got - want)[kept] - np.longdouble(2.0 ** -53) * ((9 if w is not None else 5) * size)[kept]
    assert float((error / (alpha * np.outer(norm, norm)[kept])).max()) < 2.0 ** -56.9 * (1 + -(-K // slab) if slab else 2) / 2


def test_updates_by_residues_that_are_refused(knm):
    ctx, lib = knm.default_context(), knm.load_library()
    A = torch.zeros(70, 70, device="cuda", dtype=torch.float64)
    C = torch.zeros(70, 70, device="cuda", dtype=torch.float64)

    def update(form_nt=1, n=70, k=70, slab=0, lda=70, triangular=0, ldc=70, a=A):
        return lib.precond_residue_update(ctx._h, form_nt, 0, n, k, slab, 1.0, a.data_ptr() if a is not None else None, lda, None, triangular, 0.0, 0.0,
                                          C.data_ptr(), ldc)

    assert update() == 0
    for bad in (dict(n=0), dict(k=0), dict(slab=63), dict(slab=-64), dict(slab=65600), dict(lda=69), dict(ldc=69), dict(a=None), dict(form_nt=0, triangular=1),
                dict(k=69, triangular=1)):
        assert update(**bad) == -1, bad


def test_large_fits_repeat_bit_for_bit(knm):
    n, M, d = 12_000, 6145, 9
    X, Y = _centres(n, d, 11), _centres(n, 2, 12)
    C = X[:M].contiguous()
    fits = [knm.falkon_fit(X, Y, C, 2.0, 1e-6, 4, 1e-5) for _ in range(2)]
    assert torch.equal(fits[0], fits[1])


def test_factors_on_a_card_without_room_to_spare(knm):
    """Less than a sixteenth of the card is free: the updates are fp64 products, and the factors satisfy the same identities."""
    M, d, sigma, lam, jitter = 6145, 5, 1.2, 1e-6, 1e-5
    C = _centres(M, d, M)
    free, total = torch.cuda.mem_get_info()
    others = torch.empty(max(free - total // 16 + (256 << 20), 1), device="cuda", dtype=torch.uint8)
    ctx = knm.Context()
    pre = knm.precond_build(C, sigma, lam, jitter, ctx=ctx)
    del others
    torch.cuda.empty_cache()
    T, A = _factors(pre)
    assert float((T.T @ T - _kmm(C, sigma, jitter)).abs().max()) < _bound(M)
    B = T @ T.T / M + lam * torch.eye(M, device="cuda", dtype=torch.float64)
    assert float((A.T @ A - B).abs().max()) < _bound(M) * float(B.diagonal().max())
    pre.close()
    with_room = knm.precond_build(C, sigma, lam, jitter, ctx=ctx)
    assert not torch.equal(torch.from_numpy(with_room.factors()[0]).cuda(), T)  # the other path, in the last bits
    with_room.close()
