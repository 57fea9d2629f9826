"""The routes of a2ats_score_topk against each other: the same tables and codes through two of them give
the same indices, counts and scores, bit for bit."""
import numpy as np
import pytest
import torch

from paper_2502_12665_amd import binding as B
from paper_2502_12665_amd import synth
from tests import helpers as H

pytestmark = pytest.mark.gpu


def _select(wl, xd, seq_lens, ws):
    """Tables + score/top-K with the workspace `ws`: (indices, counts, scores)."""
    st = B.DecodeState(H.dims_of(wl, xd["codes"].shape[2]), wl.top_k, wl.window, wl.n_sink, xd["q"].dtype,
                       xd["inv_freq"], wl.wrope_b)
    st.topk_idx.fill_(-7), st.topk_count.fill_(-7), st.topk_score.fill_(-7.0)
    sl = None if seq_lens is None else torch.tensor(seq_lens, dtype=torch.int32, device="cuda")
    B.build_lut(st.dims, xd["q"], st.cos_b, st.sin_b, xd["codebook"], st.q_rot, st.lut, st.lut_scale)
    B.score_topk(st.dims, xd["codes"], st.lut, st.lut_scale, wl.top_k, wl.window, wl.n_sink, sl, st.topk_idx,
                 st.topk_count, st.topk_score, None, st.ws if ws else None)
    torch.cuda.synchronize()
    return st.topk_idx, st.topk_count, st.topk_score.view(torch.int32)


@pytest.mark.parametrize("Bn,G,M,N,K,w,n_sink,lens,rows", [
    (1, 4, 16, 16384 + 300, 4096, 300, 0, None, None),                   # a quarter of the fewest candidates
    (2, 7, 32, 40001, 2049, 64, 4, None, None),                          # two head groups, the smallest wide K
    (3, 1, 16, 60000, 4096, 128, 0, [60000, 4100, 30000], None),         # sequences with few candidates more than K
    (2, 8, 16, 20000, 3000, 0, 0, [20000, 0], None),
    (1, 4, 16, 30000, 3500, 64, 4, None, "patterns"),                    # the K-th score is shared by many rows
    (1, 4, 32, 30000, 3500, 64, 4, None, "equal"),                       # every row equal: the fallback
])
def test_wide_selection_equals_the_exact_route(Bn, G, M, N, K, w, n_sink, lens, rows):
    """More than 2048 winners: the streaming route (with a workspace) against the exact route (without one)."""
    wl = synth.Workload("wide", Bn, 2 * G, 2, 128, M, N, K, w, n_sink=n_sink, seed=N + K)
    xd = synth.make_decode_inputs(wl, device="cuda", with_kv=False)
    if rows == "patterns":
        xd["codes"][:] = xd["codes"][:, :, torch.randint(0, 40, (N,), device="cuda")]
    if rows == "equal":
        xd["codes"][:] = xd["codes"][:, :, :1]
    assert B.workspace_bytes(H.dims_of(wl), B.OP_SCORE_TOPK, K, w) > 0
    for a, b in zip(_select(wl, xd, lens, True), _select(wl, xd, lens, False)):
        assert torch.equal(a, b)
