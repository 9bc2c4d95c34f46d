"""The preconditioner's symmetric updates as integer products modulo small numbers (block rows and triangular products from a few
thousand centres on): the identities that the factors satisfy, and bit-for-bit repetition.

Bound: an entry of the identities is a sum of some tens of updates, each rounded once in C (2^-53 of it) and off by at most 2^-53 of
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


# just above the size from which triangular products and then block rows are taken; tiles of 256 x 128 with remainders, several slabs of the
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


@pytest.mark.parametrize("M,weights", [(3700, "positive"), (4700, "signed"), (4500, "zeros"), (4500, "wide")])
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
