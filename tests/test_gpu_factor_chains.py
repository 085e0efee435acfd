"""The factor without blocks below the diagonal ones (half-bandwidth 0): every
64-column chunk is a chain of its own, so they run side by side.  More chunks
than there are workgroups, a last one of few columns, arrows that wait for all
of them, several failing columns, and such matrices among others in a batch.
"""
import math

import pytest

from paper_2504_19171_amd import inputs

pytestmark = pytest.mark.gpu

SHAPES = [
    # (nb, a, b)
    (64 * 700 + 5, 0, 64),
    (64 * 1100, 3, 256),
    (40001, 130, 192),
]


@pytest.mark.parametrize("nb,a,b", SHAPES)
def test_independent_chunks_match_the_oracle(oracle_mod, nb, a, b):
    import torch
    from gpu_util import factor_error, logdet_error, to_device, L_TOL, LOGDET_TOL
    from paper_2504_19171_amd import stiles as st
    M = inputs.arrowhead_spd(nb, 0, a, seed=31 + nb)
    lay = st.layout(M.n, 0, a, b)
    print(f"factor nb={nb} w=0 a={a} b={b}", flush=True)
    A = st.pack(*to_device(M, "cuda:0"), lay)
    L = torch.full_like(A, float("nan"))
    _, ld, info = st.factor(A, lay, out=L)
    torch.cuda.synchronize()
    f = oracle_mod.cholesky(M.ab, M.P, M.C)
    err, outside = factor_error(L.cpu().numpy(), lay, f, M)
    assert int(info.item()) == 0
    assert err <= L_TOL and outside == 0.0
    assert logdet_error(float(ld.item()), f) <= LOGDET_TOL


def test_first_of_several_failing_chunks():
    import torch
    from gpu_util import to_device
    from paper_2504_19171_amd import stiles as st
    M = inputs.arrowhead_spd(50000, 0, 5, seed=3)
    for bad in (49999, 1234, 30000):
        M.ab[0, bad] = -1.0
    lay = st.layout(M.n, 0, 5, 64)
    A = st.pack(*to_device(M, "cuda:0"), lay)
    _, ld, info = st.factor(A, lay, out=A)
    torch.cuda.synchronize()
    assert int(info.item()) == 1235
    assert math.isnan(float(ld.item()))


def test_in_a_batch_as_alone():
    import torch
    from gpu_util import to_device
    from paper_2504_19171_amd import stiles as st
    shapes = [(30000, 0, 0, 64), (50, 0, 7, 64), (9000, 0, 40, 128), (3000, 200, 10, 64), (500, 1, 0, 256), (64, 0, 0, 64)]
    lays, As = [], []
    for k, (nb, w, a, b) in enumerate(shapes):
        M = inputs.arrowhead_spd(nb, w, a, seed=60 + k)
        lays.append(st.layout(M.n, w, a, b))
        As.append(st.pack(*to_device(M, "cuda:0"), lays[-1]))
    Ls, ld, info = st.factor_batched(As, lays)
    torch.cuda.synchronize()
    assert int(info[:, 0].abs().max().item()) == 0
    for k, (A, lay) in enumerate(zip(As, lays)):
        L, one, _ = st.factor(A, lay)
        assert torch.equal(L.ravel(), Ls[k].ravel()), shapes[k]
        assert float(one.item()) == float(ld[k].item())


def test_chunks_run_side_by_side():
    """With w = 1 the chunks follow one another; with w = 0 they need not, which
    on hundreds of workgroups has to show."""
    import torch
    from gpu_util import to_device
    from paper_2504_19171_amd import stiles as st
    ms = {}
    for w in (0, 1):
        M = inputs.arrowhead_spd(100000, w, 0, seed=8)
        lay = st.layout(M.n, w, 0, 64)
        A = st.pack(*to_device(M, "cuda:0"), lay)
        L = torch.empty_like(A)
        ws = torch.empty(lay.factor_workspace_bytes, dtype=torch.uint8, device="cuda:0")
        times = []
        for _ in range(4):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            st.factor(A, lay, out=L, workspace=ws)
            e1.record()
            e1.synchronize()
            times.append(e0.elapsed_time(e1))
        ms[w] = min(times)
    print(f"w 0: {ms[0]:.3f} ms, w 1: {ms[1]:.3f} ms", flush=True)
    assert ms[0] < 0.25 * ms[1]
