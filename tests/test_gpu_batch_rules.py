"""Both sides of the batched calls' rules, on matrices of every tile size and
band case, bit for bit against the single calls.

Phase 2 runs with eight wavefronts a workgroup when the tile columns of the
batch together hold at most 512 tasks, else with four: every shape of the Phase
2 tests once (eight) and twice (four; each wavefront then adds two pieces of a
sum, and FAR keeps both halves of a step).  The factor takes 128 matrices a
launch, and a workgroup whose matrix is done joins another: more than that of
bands with every kind of task, of very different lengths.
"""
import pytest

from paper_2504_19171_amd import inputs
from test_gpu_phase2_blocks import SHAPES

pytestmark = pytest.mark.gpu


def _tasks(lay):
    """Phase 2 tasks of a matrix: FAR 64 x 64 blocks below tile row J + 1 and in
    the arrow, ROW and DIAG 32 x 32 blocks."""
    n64, n32, na = lay.tile // 64, lay.tile // 32, -(-lay.arrow_ld // 64)
    n = 0
    for J in range(lay.nt):
        s = min(lay.bt, lay.nt - 1 - J)
        n += (max(s - 1, 0) * n64 + na) * n64 + (n32 * n32 if s else 0) + n32 * (n32 + 1) // 2
    return n


def _compare(shapes, seed):
    import torch
    from gpu_util import to_device
    from paper_2504_19171_amd import stiles as st
    lays, As = [], []
    for k, (nb, w, a, b) in enumerate(shapes):
        M = inputs.arrowhead_spd(nb, w, a, seed=seed + k)
        lays.append(st.layout(M.n, M.w, M.a, b))
        As.append(st.pack(*to_device(M, "cuda:0"), lays[-1]))
    Ls, ld, info = st.factor_batched(As, lays)
    Ss, info = st.selinv_batched(Ls, lays, info=info)
    torch.cuda.synchronize()
    assert int(info.abs().max().item()) == 0
    for k, (A, lay) in enumerate(zip(As, lays)):
        L, one, _ = st.factor(A, lay)
        S, _ = st.selinv(L, lay)
        assert torch.equal(L.ravel(), Ls[k].ravel()), (k, shapes[k], "L")
        assert torch.equal(S.ravel(), Ss[k].ravel()), (k, shapes[k], "Sigma")
        assert float(one.item()) == float(ld[k].item()), (k, shapes[k])
    return lays


@pytest.mark.parametrize("times", [1, 2])
def test_either_number_of_wavefronts(times):
    print(f"the shapes {times} times", flush=True)
    lays = _compare(SHAPES * times, 300)
    column = sum(_tasks(lay) / lay.nt for lay in lays)
    assert (column <= 512) == (times == 1), column   # the rule's two sides


def test_several_factor_launches_of_wide_bands():
    """Widths from 3 to 6 block rows, lengths from one chunk beyond the band to
    thirty times it, with and without an arrow."""
    shapes = [(260 + 97 * (k * k % 61), 130 + 7 * (k % 36), (11 * k) % 90 if k % 3 else 0, 64) for k in range(150)]
    assert sum(-(-w // 64) >= 4 for _, w, _, _ in shapes) > 64
    print(f"batch of {len(shapes)}", flush=True)
    _compare(shapes, 1000)


def test_expired_waits_end_the_batch(monkeypatch):
    """With a spin limit of a microsecond some wait expires at once, while other
    workgroups run tasks, look for another matrix or hold a chain: every launch
    ends, every matrix reports it, and the next batch on the same buffers is
    sound."""
    import torch
    from gpu_util import to_device
    from paper_2504_19171_amd import stiles as st
    shapes = [(400 + 211 * k, 30 * k, 5 * k, 64) for k in range(1, 14)]
    lays, As = [], []
    for k, (nb, w, a, b) in enumerate(shapes):
        M = inputs.arrowhead_spd(nb, w, a, seed=2000 + k)
        lays.append(st.layout(M.n, M.w, M.a, b))
        As.append(st.pack(*to_device(M, "cuda:0"), lays[-1]))
    ws = torch.empty(st.batch_workspace_bytes(lays), dtype=torch.uint8, device="cuda:0")
    Ls = [torch.empty_like(A) for A in As]
    monkeypatch.setenv("STILES_SPIN_LIMIT_MS", "0.001")
    print("batch with a spin limit of 1 us", flush=True)
    _, ld, info = st.factor_batched(As, lays, outs=Ls, workspace=ws)
    torch.cuda.synchronize()
    assert info[:, 0].tolist() == [st.STILES_ETIMEOUT] * len(shapes)
    assert torch.isnan(ld).all()
    monkeypatch.delenv("STILES_SPIN_LIMIT_MS")
    _, ld, info = st.factor_batched(As, lays, outs=Ls, workspace=ws)
    torch.cuda.synchronize()
    assert int(info[:, 0].abs().max().item()) == 0
    for k, (A, lay) in enumerate(zip(As, lays)):
        L, one, _ = st.factor(A, lay)
        assert torch.equal(L.ravel(), Ls[k].ravel()) and float(one.item()) == float(ld[k].item()), shapes[k]
