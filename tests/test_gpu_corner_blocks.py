"""The corner: packed, factored as a dense matrix of 64 x 64 tiles, inverted by
64-column blocks.  Orders around its rules (16 rows, 64-row blocks, 512 at
most), against a dense factor in 64 bits, with the first failing column, alone
and in a batch.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

NB, W = 130, 3
ORDERS = [1, 15, 17, 64, 65, 129, 256, 257, 413, 512]


def _matrix(a, seed):
    """Band-plus-arrow input of order NB + a and the dense matrix it stands for."""
    rng = np.random.default_rng(seed)
    n = NB + a
    A = np.zeros((n, n))
    for k in range(1, W + 1):
        A[np.arange(k, NB), np.arange(NB - k)] = rng.uniform(-1, 1, NB - k)
    A[NB:, :NB] = rng.uniform(-1, 1, (a, NB)) / np.sqrt(NB)
    A[NB:, NB:] = np.tril(rng.uniform(-1, 1, (a, a)), -1) / np.sqrt(a)
    A = A + A.T
    A[np.arange(n), np.arange(n)] = 8.0 + rng.uniform(0, 1, n)
    return A


def _pack(A, a, b):
    import torch
    from paper_2504_19171_amd import stiles as st
    lay = st.layout(NB + a, W, a, b)
    ab = np.zeros((W + 1, NB))
    for k in range(W + 1):
        ab[k, :NB - k] = A[np.arange(k, NB), np.arange(NB - k)]
    d = [torch.as_tensor(np.ascontiguousarray(x), device="cuda:0") for x in (ab, A[NB:, :NB], A[NB:, NB:])]
    return lay, st.pack(*d, lay)


def _corner(T, lay):
    m = lay.arrow_ld
    return T.cpu().numpy().ravel()[-m * m:].reshape(m, m).T


@pytest.mark.parametrize("a", ORDERS)
def test_corner_factor_inverse_and_failure(a):
    from paper_2504_19171_amd import stiles as st
    A = _matrix(a, 100 + a)
    lay, T = _pack(A, a, 64)
    print(f"corner of order {a}", flush=True)
    got = _corner(T, lay)
    assert np.array_equal(got[:a, :a], A[NB:, NB:])
    assert np.array_equal(got[a:, a:], np.eye(lay.arrow_ld - a)) and not got[a:, :a].any() and not got[:a, a:].any()
    L, ld, info = st.factor(T, lay)
    assert int(info.item()) == 0
    R = np.linalg.cholesky(A)
    # rows of at most NB + a products, entries of order 3
    tol = 8.0 * (NB + a) * np.finfo(float).eps * np.linalg.cond(A)
    got = _corner(L, lay)
    assert np.abs(got[:a, :a] - R[NB:, NB:]).max() <= tol
    assert not np.triu(got, 1).any()
    assert abs(float(ld.item()) - 2 * np.log(np.diag(R)).sum()) <= tol * (NB + a)
    S, info = st.selinv(L, lay)
    assert int(info.item()) == 0
    assert np.abs(_corner(S, lay)[:a, :a] - np.linalg.inv(A)[NB:, NB:]).max() <= tol
    # the first column that fails, in the corner
    for k in sorted({0, a // 2, a - 1}):
        B = A.copy()
        B[NB + k, NB + k] = -1.0
        lay, T = _pack(B, a, 64)
        _, ld, info = st.factor(T, lay)
        assert int(info.item()) == NB + k + 1
        assert np.isnan(float(ld.item()))


def test_batch_of_corners_matches_single_calls():
    import torch
    from paper_2504_19171_amd import stiles as st
    As, lays = [], []
    for k, a in enumerate([0] + ORDERS):
        A = _matrix(a, 7 + k)
        if a == 129:
            A[NB + 100, NB + 100] = -1.0
        lay, T = _pack(A, a, (64, 128)[k % 2])
        As.append(T)
        lays.append(lay)
    print("batch of corners", flush=True)
    Ls, ld, info = st.factor_batched(As, lays)
    for k, (T, lay) in enumerate(zip(As, lays)):
        L, l1, i1 = st.factor(T, lay)
        assert int(info[k, 0].item()) == int(i1.item())
        if int(i1.item()) == 0:
            assert torch.equal(L.ravel(), Ls[k].ravel())
            assert torch.equal(l1.ravel(), ld[k:k + 1])
        else:
            assert int(i1.item()) == NB + 101 and lay.arrow == 129
