"""The persistent factor over 64 x 64 blocks (chain and left-looking tasks):
sizes at the edges of its rules, against the oracle, and the batched form
against the single calls bit for bit.

The rules change with the block half-bandwidth Wc = ceil(w / 64) (0, 1, 2, 3,
4 and more each have other tasks), with the number of chunks (fewer than the
band is wide, one, a last one with a single real column), with the arrow's
last row block (16 to 64 rows) and with the corner's groups of four chunks.
"""
import pytest

from paper_2504_19171_amd import inputs

pytestmark = pytest.mark.gpu

SHAPES = [
    # (nb, w, a, b)
    (65, 0, 0, 64),        # Wc 0, a last chunk of one column
    (640, 0, 17, 128),     # Wc 0: chunks without a block row below; arrow only
    (129, 1, 1, 64),       # Wc 1, the smallest band and arrow
    (321, 64, 64, 64),     # Wc 1 at its largest w
    (450, 65, 48, 128),    # Wc 2 at its smallest w
    (769, 128, 80, 192),   # Wc 2 at its largest w; 12 chunks and one column
    (700, 129, 16, 64),    # Wc 3
    (1025, 192, 33, 256),  # Wc 3 at its largest w
    (900, 193, 65, 64),    # Wc 4: every kind of task
    (256, 255, 20, 64),    # dense band: Wc = chunks - 1
    (1400, 500, 130, 128), # corner blocks over several groups
]


def _tensors(M):
    from gpu_util import to_device
    return to_device(M, "cuda:0")


@pytest.mark.parametrize("nb,w,a,b", SHAPES)
def test_factor_matches_oracle_at_block_edges(oracle_mod, nb, w, a, b):
    import torch
    from gpu_util import factor_error, logdet_error, L_TOL, LOGDET_TOL
    from paper_2504_19171_amd import stiles as st
    M = inputs.arrowhead_spd(nb, w, a, seed=77 + nb)
    lay = st.layout(M.n, w, a, b)
    print(f"factor nb={nb} w={w} a={a} b={b}", flush=True)
    A = st.pack(*_tensors(M), lay)
    L = torch.full_like(A, float("nan"))
    _, ld, info = st.factor(A, lay, out=L)
    torch.cuda.synchronize()
    f = oracle_mod.cholesky(M.ab, M.P, M.C)
    err, outside = factor_error(L.cpu().numpy(), lay, f, M)
    assert int(info.item()) == 0
    assert err <= L_TOL and outside == 0.0
    assert logdet_error(float(ld.item()), f) <= LOGDET_TOL


@pytest.mark.parametrize("nb,w,a,b,bad", [(900, 193, 0, 64, 0), (900, 193, 40, 128, 531), (500, 30, 5, 64, 499)])
def test_first_failing_column(nb, w, a, b, bad):
    """A diagonal entry that makes the matrix indefinite: info is its column,
    1-based, log det NaN, and the launch ends."""
    import math
    import torch
    from paper_2504_19171_amd import stiles as st
    M = inputs.arrowhead_spd(nb, w, a, seed=5)
    M.ab[0, bad] = -1.0
    lay = st.layout(M.n, w, a, b)
    A = st.pack(*_tensors(M), lay)
    _, ld, info = st.factor(A, lay, out=A)
    torch.cuda.synchronize()
    assert int(info.item()) == bad + 1
    assert math.isnan(float(ld.item()))


@pytest.mark.parametrize("cols", ["", "1", "5"])
def test_batched_factor_equals_single(monkeypatch, cols):
    """More matrices than one launch takes, of every kind of band, over several
    launches each: every L and log det as alone."""
    import torch
    from paper_2504_19171_amd import stiles as st
    if cols:
        monkeypatch.setenv("STILES_KB_COLS", cols)
    shapes = [(nb, w, a) for nb, w, a, _ in SHAPES] + [(100 + 3 * k, 5 * (k % 30), (7 * k) % 40) for k in range(125)]
    if cols:
        shapes = shapes[:16]
    lays, As = [], []
    for k, (nb, w, a) in enumerate(shapes):
        M = inputs.arrowhead_spd(nb, w, a, seed=400 + k)
        lays.append(st.layout(M.n, w, a, 64))
        As.append(st.pack(*_tensors(M), lays[-1]))
    print(f"batch of {len(As)}, cols per launch {cols or 'default'}", flush=True)
    Ls, ld, info = st.factor_batched(As, lays)
    torch.cuda.synchronize()
    assert int(info[:, 0].abs().max().item()) == 0
    for k, (A, lay) in enumerate(zip(As, lays)):
        L, one, _ = st.factor(A, lay)
        assert torch.equal(L, Ls[k]), f"matrix {k} {shapes[k]}"
        assert float(one.item()) == float(ld[k].item())
