"""Buffers that start at any double: L (and A, in place) 8 bytes past a multiple
of 16, workspaces at any byte.  The factor's loads into LDS take 16 bytes a lane
where L is aligned to them and 4 where it is not; the results are the same bit
for bit.  Sizes of every kind of task (band of 1 to many block rows, arrows of
16 to 512 rows with a last row block of every height).
"""
import pytest

from paper_2504_19171_amd import inputs

pytestmark = pytest.mark.gpu

SHAPES = [
    # (nb, w, a, b)
    (640, 0, 17, 128),
    (321, 64, 64, 64),
    (450, 65, 48, 128),
    (769, 128, 80, 192),
    (700, 129, 16, 64),
    (1025, 192, 33, 256),
    (900, 193, 65, 64),
    (1400, 500, 130, 128),
    (2000, 700, 512, 256),
]


def _packed(nb, w, a, b, seed):
    from gpu_util import to_device
    from paper_2504_19171_amd import stiles as st
    M = inputs.arrowhead_spd(nb, w, a, seed=seed)
    lay = st.layout(M.n, w, a, b)
    return lay, st.pack(*to_device(M, "cuda:0"), lay)


def _shifted(like):
    """An uninitialised buffer as long as `like`, 8 bytes past a multiple of 16."""
    import torch
    buf = torch.full((like.numel() + 1,), float("nan"), dtype=torch.float64, device=like.device)
    assert buf.data_ptr() % 16 == 0
    return buf[1:]


def _bytes(n, shift):
    import torch
    return torch.empty(n + shift, dtype=torch.uint8, device="cuda:0")[shift:]


@pytest.mark.parametrize("nb,w,a,b", SHAPES)
def test_factor_into_an_unaligned_buffer(nb, w, a, b):
    import torch
    from paper_2504_19171_amd import stiles as st
    lay, A = _packed(nb, w, a, b, 5 + nb)
    print(f"factor nb={nb} w={w} a={a} b={b}", flush=True)
    L, ld, info = st.factor(A, lay)
    out = _shifted(A)
    _, ld1, info1 = st.factor(A, lay, out=out)
    B = _shifted(A)
    B.copy_(A.ravel())
    _, ld2, info2 = st.factor(B, lay, out=B)
    torch.cuda.synchronize()
    assert int(info.item()) == int(info1.item()) == int(info2.item()) == 0
    assert torch.equal(L.ravel(), out) and torch.equal(L.ravel(), B)
    assert float(ld.item()) == float(ld1.item()) == float(ld2.item())


def test_batch_with_unaligned_buffers():
    import torch
    from paper_2504_19171_amd import stiles as st
    lays, As = zip(*[_packed(*s, 50 + k) for k, s in enumerate(SHAPES)])
    outs = [_shifted(A) if k % 2 else torch.empty_like(A) for k, A in enumerate(As)]
    _, ld, info = st.factor_batched(As, lays, outs=outs)
    torch.cuda.synchronize()
    assert int(info[:, 0].abs().max().item()) == 0
    for k, (A, lay) in enumerate(zip(As, lays)):
        L, one, _ = st.factor(A, lay)
        assert torch.equal(L.ravel(), outs[k].ravel()), SHAPES[k]
        assert float(one.item()) == float(ld[k].item())


@pytest.mark.parametrize("shift", [4, 8])
@pytest.mark.parametrize("nb,w,a,b", [(450, 65, 48, 128), (1400, 500, 130, 128)])
def test_workspaces_at_any_byte(nb, w, a, b, shift):
    import ctypes
    import torch
    from paper_2504_19171_amd import stiles as st
    lay, A = _packed(nb, w, a, b, 9 + nb)
    print(f"workspaces nb={nb} w={w} a={a} b={b} shift={shift}", flush=True)
    L, ld, _ = st.factor(A, lay)
    S, _ = st.selinv(L, lay)
    X, _ = st.inverse(L, lay)
    L1, ld1, info = st.factor(A, lay, workspace=_bytes(lay.factor_workspace_bytes, shift))
    S1, sinfo = st.selinv(L, lay, workspace=_bytes(lay.selinv_workspace_bytes, shift))
    n = int(st.load().stiles_inverse_workspace_bytes(ctypes.byref(lay._c())))
    X1, xinfo = st.inverse(L, lay, workspace=_bytes(n, shift))
    ws = _bytes(st.batch_workspace_bytes([lay, lay]), shift)
    Ls, lds, binfo = st.factor_batched([A, A], [lay, lay], workspace=ws)
    Ss, binfo = st.selinv_batched(Ls, [lay, lay], workspace=ws, info=binfo)
    torch.cuda.synchronize()
    assert int(info.item()) == int(sinfo.item()) == int(xinfo.item()) == 0
    assert int(binfo.abs().max().item()) == 0
    assert torch.equal(L, L1) and torch.equal(S, S1) and torch.equal(X, X1)
    assert float(ld.item()) == float(ld1.item())
    for k in range(2):
        assert torch.equal(Ls[k], L) and torch.equal(Ss[k], S) and float(lds[k].item()) == float(ld.item())
