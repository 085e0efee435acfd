"""Batches whose matrices share the workgroups of one launch: more matrices than
a factor launch takes (128) or than there are workgroups to share, matrices with
no tasks beside their chain, and one long matrix among short ones, which the
other workgroups join; bit for bit the single calls' results.
"""
import pytest

from paper_2504_19171_amd import inputs

pytestmark = pytest.mark.gpu


def _run(shapes):
    import torch
    from gpu_util import to_device
    from paper_2504_19171_amd import stiles as st
    lays, As = [], []
    for k, (nb, w, a, b) in enumerate(shapes):
        M = inputs.arrowhead_spd(nb, w, a, seed=900 + k)
        lay = st.layout(M.n, M.w, M.a, b)
        lays.append(lay)
        As.append(st.pack(*to_device(M, "cuda:0"), lay))
    print(f"batch of {len(shapes)}", flush=True)
    Ls, ld, info = st.factor_batched(As, lays)
    Ss, sinfo = st.selinv_batched(Ls, lays)
    assert info[:, 0].abs().max().item() == 0 and sinfo[:, 1].abs().max().item() == 0
    for k, (A, lay) in enumerate(zip(As, lays)):
        L, l1, _ = st.factor(A, lay)
        assert torch.equal(L.ravel(), Ls[k].ravel()), shapes[k]
        assert torch.equal(l1.ravel(), ld[k:k + 1]), shapes[k]
        S, _ = st.selinv(L, lay)
        assert torch.equal(S.ravel(), Ss[k].ravel()), shapes[k]


def test_more_matrices_than_workgroups():
    _run([(20 + 37 * k % 400, (3 * k) % 90, (5 * k) % 40, 64) for k in range(300)])


def test_one_long_matrix_among_short_ones():
    _run([(64, 0, 0, 64), (12000, 300, 30, 64)] + [(100 + 64 * k, 40 * k, 3 * k, (64, 128)[k % 2]) for k in range(1, 9)])
