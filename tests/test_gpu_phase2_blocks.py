"""Phase 2 of the selected inversion (FAR, ROW and DIAG tasks): sizes at the
edges of its rules, every entry of the tile pattern against a dense inverse in
64 bits, and the batched and the partial form against the single call bit for
bit.

The rules change with the tile half-bandwidth (0: no ROW; 1: no FAR rows of the
band; 2: no early rows in DIAG; 3 and more), with the part of the last band
tile that the band reaches (its sum stops there, at a multiple of 32), with the
arrow's rows (its sum of 16 k goes in steps of 32, its last row block holds 16
to 64 rows), and with the number of tile columns (none, fewer than the band is
wide, more).
"""
import numpy as np
import pytest

from paper_2504_19171_amd import inputs

pytestmark = pytest.mark.gpu

SHAPES = [
    # (nb, w, a, b)
    (60, 10, 0, 64),       # one tile column, no arrow: DIAG alone
    (300, 0, 40, 64),      # no band tiles: FAR of the arrow and DIAG
    (500, 1, 1, 64),       # the smallest band (32 rows of the last tile) and arrow
    (520, 64, 17, 64),     # bt 1, the whole last tile
    (520, 65, 80, 64),     # bt 2 at its smallest w; arrow blocks of 64 and 16 rows
    (900, 150, 0, 128),    # bt 2 without an arrow
    (900, 257, 20, 128),   # bt 3 at its smallest w
    (1000, 384, 48, 128),  # bt 3 at its largest w
    (1300, 225, 33, 192),  # a last tile reached to 225 of 384 rows
    (1500, 700, 130, 256), # bt 3, tile 256, three arrow blocks
    (700, 699, 64, 192),   # dense band: as many band tiles as columns
    (700, 500, 16, 64),    # bt 8: more columns than the first groups
]


def _factor(nb, w, a, b, seed):
    import torch  # noqa: F401  (its HIP runtime is loaded first)
    from gpu_util import to_device
    from paper_2504_19171_amd import stiles as st
    M = inputs.arrowhead_spd(nb, w, a, seed=seed)
    lay = st.layout(M.n, M.w, M.a, b)
    L, _, info = st.factor(st.pack(*to_device(M, "cuda:0"), lay), lay)
    assert int(info.item()) == 0
    return M, lay, L


def _dense(M, nb, a):
    A = np.zeros((nb + a, nb + a))
    ab = np.asarray(M.ab)
    for k in range(ab.shape[0] if ab.shape[1] == nb else ab.shape[1]):
        v = ab[k] if ab.shape[1] == nb else ab[:, k]
        A[np.arange(k, nb), np.arange(nb - k)] = v[:nb - k]
    if a:
        P = np.asarray(M.P)
        A[nb:, :nb] = P if P.shape == (a, nb) else P.T
        A[nb:, nb:] = np.tril(np.asarray(M.C))
    A = np.tril(A)
    return A + np.tril(A, -1).T


@pytest.mark.parametrize("nb,w,a,b", SHAPES)
def test_every_entry_of_the_pattern(nb, w, a, b):
    from paper_2504_19171_amd import stiles as st
    M, lay, L = _factor(nb, w, a, b, 77 + nb)
    print(f"selected inverse nb {nb} w {w} a {a} tile {b}", flush=True)
    S, info = st.selinv(L, lay)
    assert int(info.item()) == 0
    A = _dense(M, nb, a)
    X = np.linalg.inv(A)
    N, bt, ap = lay.nt * b, lay.bt, lay.arrow_ld
    F = np.eye(N)               # the padding is the identity
    F[:nb, :nb] = X[:nb, :nb]
    g = np.ones(N)
    g[:nb] = np.sqrt(np.diag(X)[:nb])
    # entries relative to sqrt(Sigma_ii Sigma_jj); rounding errors of factor
    # and inverse grow with the length of a row's sums and the condition of the
    # matrix scaled to unit diagonal
    d = 1.0 / np.sqrt(np.diag(A))
    tol = 4.0 * (w + a + 64) * np.finfo(float).eps * np.linalg.cond(A * d[:, None] * d[None, :])
    T = S.cpu().numpy().ravel()
    for J in range(lay.nt):
        c = slice(J * b, (J + 1) * b)
        for e in range(min(bt, lay.nt - 1 - J) + 1):
            r = slice((J + e) * b, (J + e + 1) * b)
            got = T[(J * (bt + 1) + e) * b * b:][:b * b].reshape(b, b).T
            err = np.abs(got - F[r, c]) / (g[r, None] * g[None, c])
            assert err.max() <= tol, (J, e, err.max(), tol)
        if a:
            m = min(b, nb - J * b)
            got = T[lay.off_arrow + J * ap * b:][:ap * b].reshape(b, ap).T[:a, :m]
            ref = X[nb:, J * b:J * b + m]
            err = np.abs(got - ref) / (np.sqrt(np.diag(X)[nb:])[:, None] * g[None, J * b:J * b + m])
            assert err.max() <= tol, (J, "arrow", err.max(), tol)


def test_batched_and_partial_forms_match_bit_for_bit():
    import torch
    from paper_2504_19171_amd import stiles as st
    fs = [_factor(*s, seed=5 + k) for k, s in enumerate(SHAPES)]
    lays, Ls = [f[1] for f in fs], [f[2] for f in fs]
    Ss, info = st.selinv_batched(Ls, lays)
    assert info[:, 1].abs().max().item() == 0
    for s, lay, L, B in zip(SHAPES, lays, Ls, Ss):
        print("batched and partial", s, flush=True)
        S, _ = st.selinv(L, lay)
        assert torch.equal(S.ravel(), B.ravel()), s
        band, arrow = lay.tile * lay.tile * (lay.bt + 1), lay.arrow_ld * lay.tile
        for jf in sorted({0, 1, lay.nt // 2, lay.nt - 1, lay.nt} & set(range(lay.nt + 1))):
            P = torch.full_like(S, float("nan"))
            P, info = st.selinv_range(L, lay, jf, out=P)
            assert int(info.item()) == 0
            assert torch.equal(P.ravel()[jf * band:lay.nt * band], S.ravel()[jf * band:lay.nt * band]), (s, jf)
            assert torch.equal(P.ravel()[lay.off_arrow + jf * arrow:], S.ravel()[lay.off_arrow + jf * arrow:]), (s, jf)


@pytest.mark.parametrize("nb,w,a,b", SHAPES + [(130, 0, 0, 64), (200, 0, 5, 64)])
def test_every_entry_of_the_inverse(nb, w, a, b):
    """The full inverse: Phase 2 over every tile below the diagonal (with w = 0
    and no arrow, sums without a term), written out in 64 x 64 blocks that end
    anywhere in the band, the arrow or both."""
    from paper_2504_19171_amd import stiles as st
    M, lay, L = _factor(nb, w, a, b, 177 + nb)
    print(f"inverse nb {nb} w {w} a {a} tile {b}", flush=True)
    X, info = st.inverse(L, lay)
    assert int(info.item()) == 0
    A = _dense(M, nb, a)
    R = np.linalg.inv(A)
    g, d = np.sqrt(np.diag(R)), 1.0 / np.sqrt(np.diag(A))
    tol = 4.0 * (w + a + 64) * np.finfo(float).eps * np.linalg.cond(A * d[:, None] * d[None, :])
    got = X.cpu().numpy().reshape(nb + a, nb + a)
    assert (np.abs(got - R) / (g[:, None] * g[None, :])).max() <= tol
    assert np.array_equal(got, got.T)
