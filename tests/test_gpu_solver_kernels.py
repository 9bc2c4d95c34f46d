"""Edges of the kernels under the preconditioner, the solves and CG: tile and group remainders, both sides of every
dispatch rule.  fp64 on both sides unless said otherwise."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def knm():
    import paper_2006_10350_amd as k

    k.load_library()
    return k


def _rand(n, d, seed):
    return torch.randn(n, d, generator=torch.Generator().manual_seed(seed)).to(torch.float32)


# one leaf with 1..8 tile rows, whole and ragged; two and three leaves
@pytest.mark.parametrize("M", [1, 15, 16, 17, 48, 100, 127, 128, 129, 144, 255, 257, 384])
def test_factors_at_leaf_edges(knm, M):
    d, sigma, lam, jitter = 6, 1.0, 1e-4, 1e-6
    C = _rand(M, d, 300 + M)
    pre = knm.precond_build(C.cuda(), sigma, lam, jitter)
    T, A = pre.factors()
    K = oracle.kernel_matrix(C.numpy(), C.numpy(), sigma) + jitter * np.eye(M)
    assert np.abs(np.tril(T, -1)).max() == 0.0
    assert np.abs(T.T @ T - K).max() < 1e-13
    assert np.abs(A.T @ A - (T @ T.T / M + lam * np.eye(M))).max() < 1e-13
    b = torch.randn(M, 2, generator=torch.Generator().manual_seed(M), dtype=torch.float64)
    got = pre.solve(b.cuda()).cpu().numpy()
    assert np.abs(A @ (T @ got) - b.numpy()).max() < 1e-9 * max(1.0, np.abs(got).max())
    pre.close()


# leaves beside the update of their rows: just below and above the size from which that is done, ragged last leaves, sub-panels within a block row
# (rows that reach back to its top), and where the update is too large for it.  Entries of K are at most 1 and of T T^T / M about that, sums of
# M products of them in fp64: 1e-13 as at the leaf's own edges.
@pytest.mark.parametrize("M", [2050, 2177, 2433, 4230, 5001])
def test_factors_with_leaves_beside_updates(knm, M):
    d, sigma, lam, jitter = 6, 1.0, 1e-4, 1e-6
    C = _rand(M, d, 300 + M).cuda()
    pre = knm.precond_build(C, sigma, lam, jitter)
    T, A = (torch.from_numpy(x).cuda() for x in pre.factors())
    c, eye = C.double(), torch.eye(M, device="cuda", dtype=torch.float64)
    r2 = torch.zeros(M, M, device="cuda", dtype=torch.float64)
    for k in range(d):
        r2 += (c[:, k, None] - c[None, :, k]) ** 2
    assert float((T.T @ T - torch.exp(-0.5 * r2 / sigma ** 2) - jitter * eye).abs().max()) < 1e-13
    assert float((A.T @ A - T @ T.T / M - lam * eye).abs().max()) < 1e-13
    pre.close()


def test_failing_pivot_inside_a_leaf(knm):
    C = _rand(300, 4, 5)
    C[171] = float("nan")  # row 171: second leaf, third tile row
    with pytest.raises(knm.KnmError) as e:
        knm.precond_build(C.cuda(), 1.0, 1e-6, 1e-6)
    assert e.value.status == -5 and "172" in str(e.value)


def test_failing_pivot_in_a_leaf_beside_an_update(knm):
    C = _rand(3000, 4, 5)
    C[171] = float("nan")
    with pytest.raises(knm.KnmError) as e:
        knm.precond_build(C.cuda(), 1.0, 1e-6, 1e-6)
    assert e.value.status == -5 and "172" in str(e.value)


# wide solve blocks: four levels of merged inverses, the last pair of a level and the last block ragged; one column,
# one and two groups of skinny products, products with wide tiles
def test_solves_with_merged_block_inverses(knm):
    M = 8501
    C = _rand(M, 12, 9)
    pre = knm.precond_build(C.cuda(), 2.0, 1e-4, 1e-5)
    T, A = (torch.from_numpy(x).cuda() for x in pre.factors())
    for t in (1, 3, 16, 21, 40):
        b = torch.randn(M, t, generator=torch.Generator().manual_seed(t), dtype=torch.float64).cuda()
        got = pre.solve(b)
        ref = torch.linalg.solve_triangular(T, torch.linalg.solve_triangular(A, b, upper=True), upper=True)
        assert float((got - ref).norm() / ref.norm()) < 1e-9, t
        got = pre.solve(b, transpose=True)
        ref = torch.linalg.solve_triangular(A.T, torch.linalg.solve_triangular(T.T, b, upper=False), upper=False)
        assert float((got - ref).norm() / ref.norm()) < 1e-9, t
    pre.close()


# more than 1024 tiles of 128 x 128: the wide tiles
@pytest.mark.parametrize("a_nt", [False, True])
def test_products_with_wide_tiles(knm, a_nt):
    g = torch.Generator(device="cuda").manual_seed(3)
    n, k = 5900, 40
    a = torch.randn(n, k, generator=g, device="cuda", dtype=torch.float64)
    A = (a.T if a_nt else a).contiguous()  # column-major n x k or k x n
    C = torch.zeros(n, n, dtype=torch.float64, device="cuda")
    knm.rank_k_update(A, C, form_nt=a_nt)
    ref = torch.triu(a @ a.T)
    assert float((C.T - ref).abs().max()) < 1e-12 * k
    ni, nj = 4230, 4200
    C = torch.zeros(nj, ni, dtype=torch.float64, device="cuda")
    knm.block_product((a[:ni].T if a_nt else a[:ni]).contiguous(), a[:nj].contiguous(), C, a_nt=a_nt)
    assert float((C.T - a[:ni] @ a[:nj].T).abs().max()) < 1e-12 * k


# 32 x 32 tiles with remainders in every direction, the last products that take them and the first that take 64 x 64 ones, also with
# operands that only allow 8-byte loads (odd leading dimensions); C is read (beta) and, with NaNs in it, not read (beta = 0)
@pytest.mark.parametrize("a_nt", [False, True])
@pytest.mark.parametrize("ni,nj,k", [(1, 1, 1), (33, 31, 7), (32, 64, 32), (95, 161, 33), (64, 65, 513), (1278, 1264, 514), (1650, 1500, 512),
                                     (1650, 1500, 514), (1651, 1701, 33)])
def test_products_with_small_tiles(knm, ni, nj, k, a_nt):
    g = torch.Generator(device="cuda").manual_seed(ni + nj + k)
    a = torch.randn(ni, k, generator=g, device="cuda", dtype=torch.float64)
    b = torch.randn(nj, k, generator=g, device="cuda", dtype=torch.float64)
    C0 = torch.randn(nj, ni, generator=g, device="cuda", dtype=torch.float64)
    ref = a @ b.T
    A = (a.T if a_nt else a).contiguous()  # column-major ni x k or k x ni
    C = C0.clone()
    knm.block_product(A, b, C, alpha=-1.0, beta=1.0, a_nt=a_nt)
    # k + 1 roundings of partial sums of products that reach about 4 each at most a few times over: far below 1e-13 (k + 10)
    assert float((C.T - (C0.T - ref)).abs().max()) < 1e-13 * (k + 10)
    C = torch.full_like(C0, float("nan"))
    knm.block_product(A, b, C, alpha=1.0, beta=0.0, a_nt=a_nt)
    assert float((C.T - ref).abs().max()) < 1e-13 * (k + 10)


# the rows' passes of sparse inputs take 16 lanes per row and walk on beyond 262144 rows: norms of rows longer than the lanes and
# of the last row, and a repeated feature found at either side of a lane group's end and in the last row
@pytest.mark.parametrize("rows,at", [(3, 15), (3, 16), (3, 32), (3, 39), (262150, 7)])
def test_csr_rows_longer_than_their_lanes(knm, rows, at):
    length = 40 if rows < 10 else 8
    d = 64
    ids = torch.arange(length).repeat(rows) + 1
    val = torch.rand(rows * length, generator=torch.Generator().manual_seed(rows + at)) + 0.5
    ptr = torch.arange(rows + 1) * length

    def csr(i):
        return torch.sparse_csr_tensor(ptr.cuda(), i.cuda(), val.cuda(), size=(rows, d), check_invariants=False)

    c_rows = 2
    C = torch.sparse_csr_tensor(ptr[:c_rows + 1].cuda(), ids[:c_rows * length].cuda(), val[:c_rows * length].cuda(), size=(c_rows, d),
                                check_invariants=False)
    V = torch.ones(c_rows, 1, device="cuda")
    _, W = knm.knm_prod_csr(csr(ids), C, 4.0, V, return_w=True)
    X64 = torch.zeros(rows, d, dtype=torch.float64)
    X64[:, 1:length + 1] = val.double().reshape(rows, length)
    K = torch.exp(-torch.cdist(X64[-3:], X64[:c_rows]) ** 2 / 32.0)
    assert float((W[-3:].cpu().double() - K.sum(1, keepdim=True)).abs().max()) < 1e-5
    bad = ids.clone()
    bad[(rows - 1) * length + at] = bad[(rows - 1) * length + at - 1]
    with pytest.raises(knm.KnmError) as e:
        knm.knm_prod_csr(csr(bad), C, 4.0, V)
    assert e.value.status == -1


def _substitute(R, b, trans):
    """Triangular solve with the upper factor R (or its transpose) in extended precision."""
    R = R.astype(np.longdouble)
    x = b.astype(np.longdouble)
    M = R.shape[0]
    for i in range(M) if trans else range(M - 1, -1, -1):
        x[i] /= R[i, i]
        if trans:
            x[i + 1:] -= np.outer(R[i, i + 1:], x[i])
        else:
            x[:i] -= np.outer(R[:i, i], x[i])
    return x


# ill-conditioned factors (the least jitters the fits are used with, and none; ratio of largest to least pivot up to 7e4).  A solve multiplies
# with the inverses of whole blocks of up to 2048, whose error bound is that of substitution times some |R^-1| |R| more; in fact the errors
# against extended precision stay within a few times those of substitution in fp64 (measured: 0.6 to 2.2)
@pytest.mark.parametrize("jitter", [1e-8, 0.0])
@pytest.mark.parametrize("M,scale", [(1000, 0.75), (2000, 2.0), (2600, 1.0), (4500, 0.75)])
def test_solves_with_ill_conditioned_factors(knm, M, scale, jitter):
    from scipy.linalg import solve_triangular

    d = 8
    pre = knm.precond_build(_rand(M, d, 500 + M).cuda(), scale * d ** 0.5, 1e-8, jitter)
    T, A = pre.factors()
    worst = {}
    for t in (1, 4):
        b = torch.randn(M, t, generator=torch.Generator().manual_seed(t), dtype=torch.float64)
        for trans in (False, True):
            first, second, op = (T, A, "T") if trans else (A, T, "N")
            exact = _substitute(second, _substitute(first, b.numpy(), trans), trans)
            plain = solve_triangular(second, solve_triangular(first, b.numpy(), trans=op), trans=op)
            got = pre.solve(b.cuda(), transpose=trans).cpu().numpy()
            worst[t, trans] = float(np.linalg.norm((got - exact).astype(float)) / np.linalg.norm((plain - exact).astype(float)))
    pre.close()
    print(f"\n  M = {M}, jitter {jitter:g}, pivot ratio {T.diagonal().max() / T.diagonal().min():.1e}: errors over substitution's",
          {k: round(v, 2) for k, v in worst.items()})
    assert max(worst.values()) < 4.0
