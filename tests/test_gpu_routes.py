"""The routes of a2ats_score_topk against each other: the same tables and codes through two of them give
the same indices, counts and scores, bit for bit."""
import threading

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


def _full_sort(wl, xd, st, seq_lens):
    """Indices, counts and scores of a full sort of the table's exact integer scores (ties by position)."""
    N, M, G, K, dev = wl.ctx_len, wl.n_sub, wl.group, wl.top_k, "cuda"
    table = st.lut[:wl.batch * wl.n_q_heads * 256 * M].reshape(wl.batch, wl.n_q_heads, 256 * M).long()
    idx = torch.full((wl.batch, wl.n_q_heads, K), -1, dtype=torch.int32, device=dev)
    cnt = torch.zeros(wl.batch, wl.n_q_heads, dtype=torch.int32, device=dev)
    score = torch.zeros(wl.batch, wl.n_q_heads, K, dtype=torch.float32, device=dev)
    for b in range(wl.batch):
        n = N if seq_lens is None else seq_lens[b]
        end = max(n - wl.window, 0)
        first = min(wl.n_sink, end)
        pos = torch.arange(first, end, device=dev)
        for h in range(wl.n_q_heads):
            at = xd["codes"][b, h // G, first:end].long() * M + torch.arange(M, device=dev)
            s = table[b, h][at].sum(1)
            best = torch.sort(s * (1 << 20) + ((1 << 20) - 1 - pos), descending=True).indices[:K]
            best = torch.sort(best).values
            k = best.numel()
            idx[b, h, :k], cnt[b, h] = (pos[best]).to(torch.int32), k
            score[b, h, :k] = s[best].to(torch.float32) * st.lut_scale[b, h]
    return idx, cnt, score.view(torch.int32)


@pytest.mark.parametrize("Bn,G,M,N,K,w,n_sink,lens,rows", [
    (2, 4, 16, 16384 + 63, 491, 63, 0, None, None),                      # the most candidates of the short route
    (1, 7, 32, 16383, 4096, 0, 4, None, None),                           # two head groups, the largest K, M = 32
    (3, 1, 16, 1025, 32, 0, 0, [1025, 1, 0], None),                      # one row past a round of the threads; one row; none
    (2, 2, 16, 3000, 3000, 16, 0, [3000, 700], None),                    # K above the candidates: all of them
    (1, 8, 16, 9000, 1, 64, 17, None, None),
    (1, 3, 16, 5000, 900, 64, 4, None, "patterns"),                      # ~125 equal scores: ties inside the band
    (2, 4, 16, 8000, 1200, 64, 4, None, "few"),                          # ~2650 equal scores: more than the band's list holds
    (33, 4, 16, 16384 + 64, 2000, 64, 0, None, "few"),
    (9, 7, 32, 5000, 4096, 0, 4, None, "few"),
    (3, 8, 16, 7001, 512, 0, 0, [7001, 2100, 1030], "few"),
    (2, 4, 32, 12000, 300, 64, 4, None, "equal"),
    (33, 4, 16, 16384 + 63, 491, 63, 0, None, None),                     # more heads than CUs: long ones by groups too
    (19, 7, 32, 16383, 4096, 0, 4, None, "patterns"),
    (33, 4, 32, 12000, 300, 64, 4, None, "equal"),                       # the band overflows: the exact route
])
def test_short_contexts_equal_a_full_sort(Bn, G, M, N, K, w, n_sink, lens, rows):
    """The short-context route (one workgroup for the heads of a group) against a full sort."""
    wl = synth.Workload("short", Bn, 2 * G, 2, 128, M, N, K, w, n_sink=n_sink, seed=N + K)
    xd = synth.make_decode_inputs(wl, device="cuda", with_kv=False)
    if rows == "patterns":
        xd["codes"][:] = xd["codes"][:, :, torch.randint(0, 40, (N,), device="cuda")]
    if rows in ("equal", "few"):
        xd["codes"][:] = xd["codes"][:, :, torch.randint(0, 3 if rows == "few" else 1, (N,), device="cuda")]
    got = _select(wl, xd, lens, True)
    st = B.DecodeState(H.dims_of(wl), K, w, n_sink, xd["q"].dtype, xd["inv_freq"], wl.wrope_b)
    B.build_lut(st.dims, xd["q"], st.cos_b, st.sin_b, xd["codebook"], st.q_rot, st.lut, st.lut_scale)
    for a, b in zip(got, _full_sort(wl, xd, st, lens)):
        assert torch.equal(a, b)


@pytest.mark.parametrize("Bn,Hkv,G,M,N,K,w,n_sink,n_new,lens,shared", [
    (2, 2, 7, 32, 9001, 300, 64, 4, 1, [9001, 2000], False),
    (40, 8, 4, 16, 1500, 45, 64, 0, 2, None, False),                     # 320 table workgroups: they encode the append
    (1, 1, 8, 32, 16384 + 128, 4096, 128, 0, 32, None, False),
    (3, 2, 8, 32, 5000, 200, 64, 4, 1, [5000, 64, 0], True),
    (2, 2, 4, 16, 6000, 0, 64, 0, 1, None, False),                       # nothing to select
    (2, 2, 4, 16, 6000, 100, 1, 0, 3, None, False),                      # two of the three appended rows are candidates
])
@pytest.mark.parametrize("rows", ["random", "few", "equal"])             # (the band overflows: tables read back by their writers)
def test_short_decode_select_equals_the_separate_calls(Bn, Hkv, G, M, N, K, w, n_sink, n_new, lens, shared, rows):
    """Append, tables and selection of a short context in one launch against the calls one after the other."""
    wl = synth.Workload("one", Bn, Hkv * G, Hkv, 128, M, N, K, w, n_sink=n_sink, seed=N)
    xd = synth.make_decode_inputs(wl, device="cuda", with_kv=False)
    if rows != "random":
        xd["codes"][:] = xd["codes"][:, :, torch.randint(0, 3 if rows == "few" else 1, (N,), device="cuda")]
    keys = synth.make_encode_keys(wl, n_new, device="cuda", stress=True)
    weights = synth.make_query_second_moment(wl)["h_diag"].cuda()
    dims, sel = H.dims_of(wl), H.dims_of(wl.replace(n_q_heads=Hkv) if shared else wl)
    sl = None if lens is None else torch.tensor(lens, dtype=torch.int32, device="cuda")
    res = []
    for fused in (True, False):
        st = B.DecodeState(dims, K, w, n_sink, xd["q"].dtype, xd["inv_freq"], wl.wrope_b)
        sk = B.DecodeState(sel, K, w, n_sink, xd["q"].dtype, xd["inv_freq"], wl.wrope_b)
        codes = xd["codes"].clone()
        for t in (st.q_rot, sk.lut, sk.lut_scale, sk.topk_idx, sk.topk_count, sk.topk_score):
            t.fill_(-7)
        tables = (xd["q"], st.cos_b, st.sin_b, xd["codebook"], st.q_rot, sk.lut, sk.lut_scale)
        pick = (K, w, n_sink, sl, sk.topk_idx, sk.topk_count, sk.topk_score)
        if fused:
            call = B.decode_select_shared if shared else B.decode_select
            call(dims, keys, n_new, N - n_new, xd["codebook"], weights, B.W_DIAG, codes, xd["q"], st.cos_b, st.sin_b,
                 st.q_rot, sk.lut, sk.lut_scale, *pick, sk.ws)
        else:
            B.encode_keys(dims, keys, n_new, N - n_new, xd["codebook"], weights, B.W_DIAG, codes, st.ws)
            (B.build_lut_shared if shared else B.build_lut)(dims, *tables)
            B.score_topk(sel, codes, sk.lut, sk.lut_scale, *pick, None, sk.ws)
        torch.cuda.synchronize()
        res.append((codes, st.q_rot, sk.lut, sk.lut_scale, sk.topk_idx, sk.topk_count, sk.topk_score))
    for a, b in zip(*res):
        assert torch.equal(a.contiguous().view(torch.uint8), b.contiguous().view(torch.uint8))


@pytest.mark.parametrize("G,Hkv,N,K,w,n_sink,dtype,page,ragged", [
    (4, 8, 700, 50, 100, 4, "bf16", 0, True),
    (7, 4, 1300, 600, 256, 0, "bf16", 16, False),                        # more rows than a staged tile; two windows' worth
    (4, 8, 300, 0, 64, 0, "f32", 0, True),                               # the window alone
    (8, 4, 513, 200, 0, 4, "f32", 64, True),                             # no window
    (8, 4, 1300, 600, 128, 0, "bf16", 16, True),
    (8, 4, 1300, 600, 128, 4, "f32", 0, False),
    (8, 4, 2600, 1500, 64, 4, "bf16", 16, True),                         # (these two: pages and lengths by the split route)
    (7, 4, 1700, 900, 100, 0, "f32", 64, True),
])
def test_attention_of_many_heads_equals_that_of_few(G, Hkv, N, K, w, n_sink, dtype, page, ragged):
    """Of many heads a workgroup of four waves takes a whole one (all cases but that with 256 window rows); the same sequences
    four at a time take a workgroup of 16 waves a head, or, with the window alone or many rows, the split route."""
    Bn = 40
    wl = synth.Workload("many", Bn, G * Hkv, Hkv, 128, 16, N, K, w, n_sink=n_sink, kv_dtype=dtype, seed=N)
    xd = synth.make_decode_inputs(wl, device="cuda")
    g = torch.Generator(device="cuda").manual_seed(N)
    lens = torch.randint(0, N + 1, (Bn,), generator=g, device="cuda", dtype=torch.int32) if ragged else None
    if ragged:
        lens[0], lens[1] = 0, 1
    k, v, table = xd["k"], xd["v"], None
    if page:
        slots = (N + page - 1) // page
        table = torch.randperm(Bn * slots, generator=g, device="cuda").reshape(Bn, slots).to(torch.int32)
        pools = []
        for x in (k, v):
            padded = torch.zeros(Bn, Hkv, slots * page, 128, dtype=x.dtype, device="cuda")
            padded[:, :, :N] = x
            pool = torch.empty(Bn * slots, Hkv, page, 128, dtype=x.dtype, device="cuda")
            pool[table.long().reshape(-1)] = (padded.reshape(Bn, Hkv, slots, page, 128).permute(0, 2, 1, 3, 4)
                                              .reshape(Bn * slots, Hkv, page, 128))
            pools.append(pool)
        k, v = pools

    def attend(first, n, idx, count):
        part = wl.replace(batch=n)
        st = B.DecodeState(H.dims_of(part), K, w, n_sink, xd["q"].dtype, xd["inv_freq"], wl.wrope_b)
        sl = None if lens is None else lens[first:first + n].contiguous()
        q = xd["q"][first:first + n].contiguous()
        q_rot = q.float().contiguous()
        st.out.fill_(7.0)
        args = (idx[first:first + n].contiguous(), count[first:first + n].contiguous(), K, w, n_sink, st.cos_win, st.sin_win,
                sl, st.out, st.ws)
        if page:
            B.sparse_attn_paged(st.dims, q, q_rot, k, v, table[first:first + n].contiguous(), page, *args)
        else:
            B.sparse_attn(st.dims, q, q_rot, k[first:first + n].contiguous(), v[first:first + n].contiguous(), *args)
        torch.cuda.synchronize()
        return st.out.float()

    heads = G * Hkv
    idx = torch.sort(torch.rand(Bn, heads, max(N - w, 1), generator=g, device="cuda").argsort(-1)[..., :max(K, 1)], -1).values
    idx = idx.to(torch.int32)
    count = torch.full((Bn, heads), K, dtype=torch.int32, device="cuda")
    whole = attend(0, Bn, idx, count)
    few = torch.cat([attend(b, 4, idx, count) for b in range(0, Bn, 4)])
    # float32 sums in another order, 4e-6 of the values' size (about 1); a bfloat16 output may round the other way, and
    # neighbours of 8 significant bits are up to 2^-7 of themselves apart
    tol = 2.0 ** -7 if dtype == "bf16" else 4e-6
    assert ((whole - few).abs() <= tol * torch.maximum(whole.abs(), few.abs()) + 4e-6).all(), float((whole - few).abs().max())


@pytest.mark.parametrize("Bn,G,M,N,K,n_sink", [
    (2, 4, 16, 12000, 300, 4),        # the exact route, its keys in registers
    (1, 4, 32, 12000, 300, 0),
    (2, 4, 16, 40000, 4000, 4),       # without a workspace the exact route, its keys scored again and again
    (40, 4, 16, 12000, 300, 4),       # a workgroup per group
    (2, 4, 16, 60000, 1500, 4),       # the streaming route
    (42, 4, 16, 20000, 600, 4),       # lists of a workgroup per group
])
@pytest.mark.parametrize("bad", ["inf", "nan", "huge"])
def test_queries_that_are_not_finite_select_within_their_rows(Bn, G, M, N, K, n_sink, bad):
    """Table entries of an infinite query saturate and their sums wrap.  What is selected then means nothing, but it is K'
    ascending candidates per head, and nothing is written anywhere else."""
    wl = synth.Workload("bad", Bn, 2 * G, 2, 128, M, N, K, 64, n_sink=n_sink, seed=N + K)
    xd = synth.make_decode_inputs(wl, device="cuda", with_kv=False)
    q = xd["q"].float()
    if bad == "huge":
        q *= 3e38
    else:
        q[:, ::2, 5] = float(bad)
        q[:, 1, 64:] = -float(bad)
        q[-1, -1, ::3] = float(bad)
    dims = H.dims_of(wl)
    st = B.DecodeState(dims, K, 64, n_sink, torch.float32, xd["inv_freq"], wl.wrope_b)
    heads = Bn * 2 * G
    idx = torch.full((heads * K + N,), -7, dtype=torch.int32, device="cuda")
    score = torch.full((heads * K + N,), -7.0, device="cuda")
    B.build_lut(dims, q, st.cos_b, st.sin_b, xd["codebook"], st.q_rot, st.lut, st.lut_scale)
    for ws in (st.ws, None) if K > 2048 else (st.ws,):
        B.score_topk(dims, xd["codes"], st.lut, st.lut_scale, K, 64, n_sink, None, idx, st.topk_count, score, None, ws)
        torch.cuda.synchronize()
        assert (idx[heads * K:] == -7).all() and (score[heads * K:] == -7.0).all()
        assert (st.topk_count == K).all()
        got = idx[:heads * K].view(heads, K)
        assert (got[:, 1:] > got[:, :-1]).all() and (got >= n_sink).all() and (got < N - 64).all()


@pytest.mark.parametrize("Bn,G,Hkv,M,N,K,w,n_sink", [
    (1, 4, 2, 16, 3000, 300, 64, 4),      # a workgroup per head
    (2, 3, 2, 32, 16384 + 64, 700, 64, 0),
    (16, 4, 8, 16, 3000, 300, 64, 4),     # by group
    (2, 4, 2, 16, 40000, 1200, 64, 4),    # the streaming route
    (40, 8, 2, 32, 20000, 600, 64, 0),    # ... with one sampling workgroup a problem
    (1, 4, 1, 1, 20000, 500, 64, 4),      # a single codebook: one head a workgroup
    (5, 7, 2, 1, 9000, 4000, 64, 0),      # (and more than four vectors of a KV head)
    (40, 4, 2, 1, 40000, 500, 64, 0),     # two heads, longer chunks
])
@pytest.mark.parametrize("bad", ["inf", "nan", "huge"])
def test_decode_select_of_values_that_are_not_finite_equals_the_two_calls(Bn, G, Hkv, M, N, K, w, n_sink, bad):
    """Queries and appended keys that are not finite through the one call: tables, codes and counts of the two calls, bit for bit,
    K' ascending candidates per head, and nothing behind the outputs.  (Which candidates is told by the single codebook only,
    whose scores are table entries; the sums of the others wrap, and the routes order them differently.)"""
    wl = synth.Workload("bad", Bn, Hkv * G, Hkv, 128, M, N, K, w, n_sink=n_sink, seed=N + K,
                        n_centroids=4096 if M == 1 else 256)
    xd = synth.make_decode_inputs(wl, device="cuda", with_kv=False)
    q, keys = xd["q"].float(), synth.make_encode_keys(wl, 1, device="cuda")
    if bad == "huge":
        q *= 3e38
        keys[::2] *= 1e38
    else:
        q[:, ::2, 5] = float(bad)
        q[:, 1, 64:] = -float(bad)
        q[-1, -1, ::3] = float(bad)
        keys[0, :, :, 7] = float(bad)
        keys[-1, -1, :, 70:] = -float(bad)
    dims = H.dims_of(wl)
    heads = Bn * Hkv * G
    ws = torch.empty(max(B.workspace_bytes(dims, B.OP_ENCODE), B.workspace_bytes(dims, B.OP_SCORE_TOPK, K, w), 256),
                     dtype=torch.uint8, device="cuda")
    res = []
    for one in (False, True):
        st = B.DecodeState(dims, K, w, n_sink, torch.float32, xd["inv_freq"], wl.wrope_b)
        st.lut.fill_(-1)
        idx = torch.full((heads * K + N,), -7, dtype=torch.int32, device="cuda")
        score = torch.full((heads * K + N,), -7.0, device="cuda")
        codes = torch.cat([xd["codes"].reshape(-1), xd["codes"].reshape(-1)[:256]])
        args = (dims, keys, 1, N - 1, xd["codebook"], None, B.W_NONE, codes, q, st.cos_b, st.sin_b, st.q_rot, st.lut,
                st.lut_scale)
        if one:
            B.decode_select(*args, K, w, n_sink, None, idx, st.topk_count, score, ws)
        else:
            B.decode_prologue(*args, ws)
            B.score_topk(dims, codes, st.lut, st.lut_scale, K, w, n_sink, None, idx, st.topk_count, score, None, ws)
        torch.cuda.synchronize()
        res.append([t.view(torch.int32) for t in (st.lut, st.lut_scale, st.q_rot, st.topk_count)] + [codes] +
                   ([idx, score.view(torch.int32)] if M == 1 else []))
        assert (idx[heads * K:] == -7).all() and (score[heads * K:] == -7.0).all()
        assert torch.equal(codes[-256:], xd["codes"].reshape(-1)[:256])
        got = idx[:heads * K].view(heads, K)
        assert (st.topk_count == K).all()
        assert (got[:, 1:] > got[:, :-1]).all() and (got >= n_sink).all() and (got < N - w).all()
    for a, b in zip(*res):
        assert torch.equal(a, b)


@pytest.mark.parametrize("N,K,w,n_sink", [(700, 100, 64, 4), (700, 508, 100, 0), (5000, 4096, 64, 4), (1500, 1000, 0, 0), (900, 0, 230, 0)])
def test_float32_attention_of_many_heads_is_as_exact_as_that_of_few(N, K, w, n_sink):
    """The same four sequences among 40 (a workgroup of four waves takes a whole head) and alone (its rows are shared out; the
    first two cases: taken by 16 waves), against float64: errors of rounding only, and of the same size."""
    Bn, Hkv, G, n = 40, 4, 8, 4
    wl = synth.Workload("exact", Bn, Hkv * G, Hkv, 128, 16, N, K, w, n_sink=n_sink, kv_dtype="f32", seed=N)
    xd = synth.make_decode_inputs(wl, device="cuda")
    g = torch.Generator(device="cuda").manual_seed(N)
    idx = torch.rand(Bn, Hkv * G, N - w - n_sink, generator=g, device="cuda").topk(max(K, 1), -1).indices
    idx = (torch.sort(idx, -1).values + n_sink).to(torch.int32).contiguous()
    count = torch.full((Bn, Hkv * G), K, dtype=torch.int32, device="cuda")
    outs = []
    for take in (Bn, n):
        st = B.DecodeState(H.dims_of(wl.replace(batch=take)), K, w, n_sink, torch.float32, xd["inv_freq"], wl.wrope_b)
        B.sparse_attn(st.dims, xd["q"][:take], xd["q"][:take], xd["k"][:take], xd["v"][:take], idx[:take], count[:take], K, w,
                      n_sink, st.cos_win, st.sin_win, None, st.out, st.ws)
        torch.cuda.synchronize()
        outs.append(st.out[:n].double())
    back = torch.arange(w - 1, -1, -1, device="cuda")
    cos, sin = st.cos_win.double()[back], st.sin_win.double()[back]
    err, size = [0.0, 0.0], 0.0
    for b in range(n):
        for h in range(Hkv * G):
            k, v, q = xd["k"][b, h // G].double(), xd["v"][b, h // G].double(), xd["q"][b, h].double()
            far = torch.cat([torch.arange(n_sink, device="cuda"), idx[b, h, :K].long()])
            turned = torch.cat([q[:64] * cos - q[64:] * sin, q[64:] * cos + q[:64] * sin], 1)
            logit = torch.cat([k[far] @ q, (turned * k[N - w:]).sum(1)]) * 128 ** -0.5
            want = torch.softmax(logit, 0) @ torch.cat([v[far], v[N - w:]])
            size += float(want.pow(2).sum())
            for i, o in enumerate(outs):
                err[i] += float((o[b, h] - want).pow(2).sum())
    whole, few = (err[0] / size) ** 0.5, (err[1] / size) ** 0.5
    H.log(f"float32 attention, {K} + {w} rows: error {whole:.3e} of many heads, {few:.3e} of few")
    assert whole <= 1.1 * few and few < 4e-7


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("Bn,G,Hkv,N,K,w,n_sink,lens", [
    (1, 4, 1, 500, 1, 1, 0, None),                    # a row of each kind
    (2, 7, 2, 900, 336, 60, 4, [900, 3]),             # the most rows of few heads; a sequence shorter than its window
    (3, 8, 4, 2500, 680, 120, 0, [2500, 70, 1]),      # the most of 96 (float32); no candidates
    (16, 4, 4, 1000, 30, 131, 4, None),               # 256 heads; window rows the most
    (3, 8, 4, 2500, 1140, 56, 4, None),               # the most of bf16
    (2, 4, 2, 600, 100, 0, 0, None),                  # no window
    (1, 4, 1, 500, 1, 70, 0, None),                   # (this and the next ones within attn_block's limits of their head counts)
    (2, 7, 2, 900, 296, 100, 4, [900, 3]),
    (18, 8, 1, 600, 100, 0, 0, None),
    (24, 4, 1, 300, 1, 64, 0, None),
    (5, 8, 4, 2500, 1140, 56, 4, [2500, 60, 1, 0, 1200]),
    (5, 8, 4, 1000, 400, 236, 4, [1000, 700, 200, 0, 1]),
    (22, 8, 1, 2500, 1140, 56, 4, None),
])
def test_attention_of_few_rows_by_one_workgroup(Bn, G, Hkv, N, K, w, n_sink, lens, dtype):
    """Few rows a head: a workgroup of 16 waves takes them all.  Against float64; other sequences of the batch do not matter."""
    wl = synth.Workload("block", Bn, Hkv * G, Hkv, 128, 16, N, K, w, n_sink=n_sink, kv_dtype=dtype, seed=N + K)
    xd = synth.make_decode_inputs(wl, device="cuda")
    g = torch.Generator(device="cuda").manual_seed(N)
    lens = lens or [N] * Bn
    idx = torch.zeros(Bn, Hkv * G, K, dtype=torch.int32, device="cuda")
    count = torch.zeros(Bn, Hkv * G, dtype=torch.int32, device="cuda")
    for b, n in enumerate(lens):
        start = max(n - w, 0)
        c = max(min(K, start - n_sink), 0)
        if c:
            pick = torch.rand(Hkv * G, start - n_sink, generator=g, device="cuda").topk(c, -1).indices
            idx[b, :, :c] = (torch.sort(pick, -1).values + n_sink).to(torch.int32)
        count[b] = c
    st = B.DecodeState(H.dims_of(wl), K, w, n_sink, xd["q"].dtype, xd["inv_freq"], wl.wrope_b)
    st.out.fill_(7.0)
    B.sparse_attn(st.dims, xd["q"], xd["q"].float().contiguous(), xd["k"], xd["v"], idx, count, K, w, n_sink, st.cos_win,
                  st.sin_win, torch.tensor(lens, dtype=torch.int32, device="cuda"), st.out, st.ws)
    torch.cuda.synchronize()
    # a bfloat16 output has 8 significant bits; float32: 1200 products and sums of values of size 1
    tol = 2.0 ** -8 if dtype == "bf16" else 2e-6
    for b, n in enumerate(lens):
        start = max(n - w, 0)
        back = torch.arange(n - start - 1, -1, -1, device="cuda")
        cos, sin = st.cos_win.double()[back], st.sin_win.double()[back]
        for h in range(Hkv * G):
            k, v, q = xd["k"][b, h // G].double(), xd["v"][b, h // G].double(), xd["q"][b, h].double()
            far = torch.cat([torch.arange(min(n_sink, start), device="cuda"), idx[b, h, :int(count[b, h])].long()])
            turned = torch.cat([q[:64] * cos - q[64:] * sin, q[64:] * cos + q[:64] * sin], 1)
            logit = torch.cat([k[far] @ q, (turned * k[start:n]).sum(1)]) * 128 ** -0.5
            want = torch.softmax(logit, 0) @ torch.cat([v[far], v[start:n]])
            got = st.out[b, h].double()
            assert ((got - want).abs() <= tol * want.abs() + 2e-6).all(), (b, h, float((got - want).abs().max()))


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("Hkv,K,w", [(8, 100, 64), (32, 100, 66), (96, 100, 1), (48, 200, 100)])
def test_attention_of_few_rows_by_one_workgroup_of_values_that_are_not_finite(Hkv, K, w, dtype):
    """A row whose logit is -inf has no weight, wherever a wave meets it (alone, first, last, at both ends of a link); a logit
    that is not a number empties its own head alone, and what is not finite among the values stays in its dimension."""
    N = K + w
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    g = torch.Generator(device="cuda").manual_seed(N)
    k, v = (torch.randn(1, Hkv, N, 128, generator=g, device="cuda").to(dt) for _ in range(2))
    q = torch.ones(1, Hkv, 128, dtype=dt, device="cuda")
    dims = B.make_dims(1, Hkv, Hkv, 128, 16, N)
    st = B.DecodeState(dims, K, w, 0, dt, synth.inv_freq(128, 10000.0), 1)
    idx = torch.arange(K, dtype=torch.int32, device="cuda").expand(1, Hkv, K).contiguous()
    count = torch.full((1, Hkv), K, dtype=torch.int32, device="cuda")
    inf = float("inf")
    # (dimension 63 turns the least: its factor is positive at every distance)
    lost = torch.zeros(Hkv, N, dtype=torch.bool, device="cuda")
    lost[0, N - 1] = lost[1, 0] = lost[2, K - 1] = True
    lost[3, K:] = lost[4, :K] = True
    lost[5, :64] = lost[5, K:K + w // 2] = True
    lost[7] = torch.rand(N, generator=g, device="cuda") < 0.5
    k[0, :, :, 63] = torch.where(lost, -inf, k[0, :, :, 63].float()).to(dt)
    k[0, 6, 5, 63] = float("nan")
    v[0, 7, int((~lost[7]).nonzero()[0]), 9] = inf
    B.sparse_attn(dims, q, q.float().contiguous(), k, v, idx, count, K, w, 0, st.cos_win, st.sin_win, None, st.out, st.ws)
    torch.cuda.synchronize()
    back = torch.arange(w - 1, -1, -1, device="cuda")
    cos, sin = st.cos_win.double()[back], st.sin_win.double()[back]
    turn = torch.cat([torch.ones(K, 128, dtype=torch.float64, device="cuda"), torch.cat([cos - sin, cos + sin], 1)])
    tol = 2.0 ** -8 if dtype == "bf16" else 2e-6   # (as above)
    for h in range(Hkv):
        if h == 6:
            assert (st.out[0, h] == 0).all()
            continue
        logit = (turn * torch.where(lost[h][:, None], 0.0, k[0, h].double())).sum(1) * 128 ** -0.5
        want = torch.softmax(torch.where(lost[h], -inf, logit), 0) @ torch.where(lost[h][:, None], 0.0, v[0, h].double())
        got, fine = st.out[0, h].double(), torch.ones(128, dtype=torch.bool, device="cuda")
        if h == 7:
            fine[9] = False
            assert got[9] == inf
        assert ((got - want).abs() <= tol * want.abs() + 2e-6)[fine].all(), (h, float((got - want).abs()[fine].max()))


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("Hkv,K,w", [(1, 16, 16), (2, 0, 16), (64, 256, 100), (128, 64, 64)])
def test_attention_over_an_empty_context_gives_zeros(Hkv, K, w, dtype):
    """ctx_len = 0 in a cache that has room for more, through every per-head call."""
    heads = 4 * Hkv
    cache = torch.ones(1, Hkv, 32, 128, dtype=torch.float32 if dtype == "f32" else torch.bfloat16, device="cuda")
    dims = B.make_dims(1, heads, Hkv, 128, 16, 0, 32)
    st = B.DecodeState(dims, K, w, 0, cache.dtype, synth.inv_freq(128, 10000.0), 1)
    q = torch.ones(1, heads, 128, dtype=cache.dtype, device="cuda")
    q_rot = q.float().contiguous()
    idx = torch.zeros(1, heads, max(K, 1), dtype=torch.int32, device="cuda")
    count = torch.full((1, heads), K, dtype=torch.int32, device="cuda")
    pool, table = cache.reshape(1, Hkv, 2, 16, 128).transpose(1, 2).reshape(2, Hkv, 16, 128).contiguous(), torch.tensor(
        [[0, 1]], dtype=torch.int32, device="cuda")
    tail = (idx, count, K, w, 0, st.cos_win, st.sin_win, None, st.out)
    for call in (lambda: B.sparse_attn(dims, q, q_rot, cache, cache, *tail, st.ws),
                 lambda: B.sparse_attn_static(dims, q, q_rot, cache, cache, *tail),
                 lambda: B.sparse_attn_paged(dims, q, q_rot, pool, pool, table, 16, *tail, st.ws)):
        st.out.fill_(7.0)
        call()
        torch.cuda.synchronize()
        assert (st.out == 0).all()


@pytest.mark.parametrize("Bn,G,Hkv,N,K,w,n_sink,n_new,lens,stride,data", [
    (1, 4, 1, 4096 + 16, 100, 16, 0, 1, None, 0, None),          # one head a workgroup, exactly one chunk of 4096
    (1, 4, 1, 4097 + 16, 100, 16, 0, 2, None, 8, None),          # and one token more
    (2, 7, 2, 9000, 777, 32, 4, 1, [9000, 4104], 5, None),       # rows that do not start on 16 bytes; an odd group
    (2, 8, 2, 50000, 4096, 64, 3, 8, None, 0, "patterns"),       # the K-th score is shared by many tokens
    (3, 4, 8, 70001, 1500, 128, 4, 1, [70001, 1, 33000], 7, None),   # two heads a workgroup, sequences without candidates
    (33, 4, 8, 17000, 600, 64, 0, 1, None, 0, None),             # four heads a workgroup, two chunks of 16384
    (17, 7, 8, 16500, 300, 64, 1, 1, [16500] * 16 + [360], 0, "patterns"),   # of which the last has three; everything selected
    (1, 1, 2, 20000, 3000, 64, 0, 1, None, 0, "equal"),          # a table of equal scores: radix levels, lowest positions
    (4, 4, 2, 12000, 3999, 64, 4, 3, None, 0, "crowded"),        # nearly equal scores: a crowded bin
    (2, 4, 1, 700, 636, 64, 0, 1, None, 0, None),                # few tokens: the counts do not fit, the two calls
    (1, 2, 1, 6000, 0, 64, 0, 1, None, 0, None),
    (40, 1, 8, 140000, 1000, 64, 4, 1, None, 0, None),           # too many chunks of too many heads: the two calls
    (36, 1, 8, 49152 + 68, 1000, 64, 4, 1, None, 0, None),       # the most that still go by chunk, exactly three of them
])
@pytest.mark.parametrize("mode", ["none", "block"])
def test_single_codebook_decode_select_equals_the_two_calls(Bn, G, Hkv, N, K, w, n_sink, n_new, lens, stride, data, mode):
    """Tables, appended keys and selection from counts in two launches against prologue and selection as calls of their own:
    every output bit for bit; no memory behind the outputs is written."""
    wl = synth.Workload("single_select", Bn, G * Hkv, Hkv, 128, 1, N, K, w, n_sink=n_sink, n_centroids=4096, seed=N + K)
    xd = synth.make_decode_inputs(wl, device="cuda", with_kv=False)
    if data == "patterns":
        xd["codes"][:] = xd["codes"][:, :, torch.randint(0, 60, (N,), device="cuda")]
    if data == "equal":
        xd["codebook"][:] = xd["codebook"][:, :, :1]
    if data == "crowded":
        xd["codebook"][:, :, 1:3000] = xd["codebook"][:, :, :1] * (1 + 1e-6 * torch.rand(2999, 1, device="cuda"))
        xd["codebook"][:, :, 500:900] = xd["codebook"][:, :, :1]
    weights = None if mode == "none" else synth.make_query_second_moment(wl)["h_block"].cuda()
    wmode = B.W_NONE if mode == "none" else B.W_BLOCK
    keys = synth.make_encode_keys(wl, n_new, device="cuda", stress=True)
    dims = H.dims_of(wl, N + stride)
    full = torch.zeros(Bn, Hkv, N + stride, 1, dtype=xd["codes"].dtype, device="cuda")
    full[:, :, :N] = xd["codes"]
    sl = None if lens is None else torch.tensor(lens, dtype=torch.int32, device="cuda")
    ws = torch.empty(B.workspace_bytes(dims, B.OP_ENCODE), dtype=torch.uint8, device="cuda")
    res = []
    for how in ("two calls", "one", "one, prepared"):
        st = B.DecodeState(dims, max(K, 1), w, n_sink, xd["q"].dtype, xd["inv_freq"], wl.wrope_b)
        st.lut.fill_(-1)
        idx = torch.full((Bn * Hkv * G * K + 8,), -7, dtype=torch.int32, device="cuda")
        score = torch.full((Bn * Hkv * G * K + 8,), -7.0, device="cuda")
        codes = full.clone()
        ws.fill_(255)
        flag = 0
        if how == "one, prepared":
            B.encode_prepare(dims, xd["codebook"], weights, wmode, ws)
            flag = B.W_PREPARED
        args = (dims, keys, n_new, N - n_new, xd["codebook"], weights, wmode | flag, codes, xd["q"], st.cos_b, st.sin_b,
                st.q_rot, st.lut, st.lut_scale)
        if how == "two calls":
            B.decode_prologue(*args, ws)
            B.score_topk(dims, codes, st.lut, st.lut_scale, K, w, n_sink, sl, idx, st.topk_count, score, None, None)
        else:
            B.decode_select(*args, K, w, n_sink, sl, idx, st.topk_count, score, ws)
        torch.cuda.synchronize()
        res.append((codes, st.lut, st.lut_scale, st.q_rot, idx, st.topk_count, score.view(torch.int32)))
    for other in res[1:]:
        for a, b in zip(res[0], other):
            assert torch.equal(a, b)
    assert (res[1][4][-8:] == -7).all() and (res[1][0][:, :, N:] == 0).all()


@pytest.mark.parametrize("Bn,Hkv,n_new", [(1, 1, 1), (1, 8, 1), (1, 4, 4), (1, 2, 5), (4, 8, 1), (5, 3, 1), (3, 2, 8), (17, 1, 1)])
@pytest.mark.parametrize("mode", ["none", "diag", "block"])
def test_single_codebook_keys_between_two_codewords_get_one_code_from_every_call(Bn, Hkv, n_new, mode):
    """Keys half way between their two nearest codewords, so that only the rounding of the distortions tells these apart:
    the calls that append keys agree, whatever the number of keys and whichever sweep that takes."""
    g = torch.Generator(device="cuda").manual_seed(Bn * 64 + Hkv * 8 + n_new)
    N, n = 4096 + 100, Bn * n_new
    keys = torch.round(torch.randn(Bn, Hkv, n_new, 128, generator=g, device="cuda") * 512) / 512
    codebook = torch.randn(Hkv, 4096, 128, generator=g, device="cuda") * 8
    at = torch.stack([torch.randperm(4096, generator=g, device="cuda")[:2 * n] for _ in range(Hkv)])
    for h in range(Hkv):
        k = keys[:, h].reshape(n, 128)
        off = torch.round(torch.randn(n, 128, generator=g, device="cuda") * 64) / 512   # (sums exact in float32)
        codebook[h, at[h, :n]], codebook[h, at[h, n:]] = k + off, k - off
    codebook = codebook.reshape(Hkv, 1, 4096, 128).contiguous()
    a = torch.randn(Hkv, 128, 128, generator=g, device="cuda")
    weights = {"none": None, "diag": torch.rand(Hkv, 128, generator=g, device="cuda") + 0.5,
               "block": (torch.matmul(a, a.transpose(1, 2).contiguous()) / 128 + torch.eye(128, device="cuda")).contiguous()}[mode]
    wmode = {"none": B.W_NONE, "diag": B.W_DIAG, "block": B.W_BLOCK}[mode]
    q = torch.randn(Bn, 2 * Hkv, 128, generator=g, device="cuda")
    inv = torch.tensor([1e4 ** (-i / 64) for i in range(64)], dtype=torch.float64)
    res = []
    for how in ("encode", "prologue", "select", "one sequence at a time", "one key at a time"):
        codes = torch.zeros(Bn, Hkv, N, 1, dtype=torch.int16, device="cuda")
        step = 1 if how == "one sequence at a time" else Bn
        for b in range(0, Bn, step):
            dims = B.make_dims(step, 2 * Hkv, Hkv, 128, 1, N, n_centroids=4096)
            st = B.DecodeState(dims, 64, 64, 0, torch.float32, inv, 100)
            ws = torch.empty(B.workspace_bytes(dims, B.OP_ENCODE), dtype=torch.uint8, device="cuda")
            part = codes[b:b + step]
            args = (part, q[b:b + step], st.cos_b, st.sin_b, st.q_rot, st.lut, st.lut_scale)
            new = keys[b:b + step].contiguous()
            if how in ("encode", "one sequence at a time"):
                B.encode_keys(dims, new, n_new, N - n_new, codebook, weights, wmode, part, ws)
            elif how == "one key at a time":
                for j in range(n_new):
                    B.encode_keys(dims, new[:, :, j:j + 1].contiguous(), 1, N - n_new + j, codebook, weights, wmode, part, ws)
            elif how == "prologue":
                B.decode_prologue(dims, new, n_new, N - n_new, codebook, weights, wmode, *args, ws)
            else:
                B.decode_select(dims, new, n_new, N - n_new, codebook, weights, wmode, *args, 64, 64, 0, None, st.topk_idx,
                                st.topk_count, None, ws)
            torch.cuda.synchronize()
        res.append(codes)
    got = res[0][:, :, N - n_new:, 0].long()
    pair = at.reshape(Hkv, 2, Bn, n_new)
    assert ((got == pair[:, 0].transpose(0, 1)) | (got == pair[:, 1].transpose(0, 1))).all()
    for other in res[1:]:
        assert torch.equal(res[0], other)


@pytest.mark.parametrize("Bn,G,Hkv", [(5, 1, 2), (4, 2, 1), (3, 4, 3), (2, 7, 1), (17, 1, 1), (1, 8, 1)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("shared", [False, True])
def test_single_codebook_tables_of_few_heads_equal_those_of_many(Bn, G, Hkv, dtype, shared):
    """One to four vectors of a KV head take smaller products in more workgroups: the same tables bit for bit, and those
    of float64 sums rounded once."""
    g = torch.Generator(device="cuda").manual_seed(Bn * 8 + G)
    codebook = torch.randn(Hkv, 1, 4096, 128, generator=g, device="cuda")
    q = torch.randn(Bn, Hkv * G, 128, generator=g, device="cuda").to(dtype)
    cos, sin, _, _ = B.rope_tables(128, torch.tensor([1e4 ** (-i / 64) for i in range(64)], dtype=torch.float64), 33, 4, "cuda")
    heads = Hkv if shared else Hkv * G

    def tables(q):
        n = q.shape[0]
        dims = B.make_dims(n, Hkv * G, Hkv, 128, 1, 64, n_centroids=4096)
        lut = torch.full((n * heads * 4096 + 64,), -7, dtype=torch.int32, device="cuda")
        q_rot, scale = torch.empty(n, Hkv * G, 128, device="cuda"), torch.zeros(n, heads, device="cuda")
        (B.build_lut_shared if shared else B.build_lut)(dims, q.contiguous(), cos, sin, codebook, q_rot, lut, scale)
        torch.cuda.synchronize()
        assert (lut[n * heads * 4096:] == -7).all() and (scale == 1).all()
        return lut[:n * heads * 4096].reshape(n, heads, 4096), q_rot

    lut, q_rot = tables(q)
    for b in range(Bn):
        one = tables(q[b:b + 1])
        assert torch.equal(one[0][0], lut[b]) and torch.equal(one[1][0], q_rot[b])
    v = q_rot.double().reshape(Bn, Hkv, G, 128)
    if shared:
        v = v.sum(2, keepdim=True).float().double()
    want = torch.matmul(v, codebook.double().reshape(1, Hkv, 4096, 128).transpose(2, 3).contiguous()).reshape(Bn, heads, 4096)
    got = torch.where(lut < 0, lut ^ 0x7FFFFFFF, lut).view(torch.float32).double()
    # half an ulp of float32; float64 sums of 128 products in two orders, of magnitudes that add up to some 80
    assert ((got - want).abs() <= 6e-8 * want.abs() + 1e-12).all()


@pytest.mark.parametrize("Bn,G,Hkv,M,N,K,w,n_sink,n_new,lens,data", [
    (1, 1, 1, 16, 40, 7, 32, 4, 1, None, None),                       # four candidates
    (2, 3, 2, 32, 1024 + 64, 300, 64, 0, 1, None, None),              # one row a thread, exactly; a group of three
    (2, 4, 2, 16, 1025 + 64, 300, 64, 0, 2, [1089, 64], None),        # and one row more; a sequence without candidates
    (3, 7, 2, 32, 16384 + 68, 4096, 64, 4, 1, [16452, 0, 9000], None),   # the most candidates; a second group of three
    (3, 7, 2, 16, 16383 + 64, 2000, 64, 0, 1, None, "patterns"),      # the K-th score is shared by many rows
    (1, 8, 1, 16, 9000, 8000 // 2, 64, 0, 1, None, "equal"),          # every row equal
    (2, 5, 1, 32, 700, 700, 64, 2, 3, None, None),                    # everything selected
    (1, 4, 2, 16, 3000, 0, 64, 0, 1, None, None),                     # nothing
    (8, 4, 8, 32, 2000, 100, 64, 0, 1, None, None),                   # 256 heads: they encode the keys as well
    (8, 4, 8, 32, 2000, 100, 64, 0, 8, None, None),                   # too many keys for that: by group
    (8, 4, 8, 32, 2000, 100, 64, 0, 16, None, None),                  # neither leaves room for workgroups that encode
    (8, 4, 8, 16, 9000, 500, 64, 4, 4, None, "zero"),                 # the same; queries of zero
    (33, 1, 8, 16, 2500, 100, 64, 0, 1, None, None),                  # 264 groups of one head, in two rounds
])
@pytest.mark.parametrize("shared", [False, True])
def test_selection_by_head_equals_the_calls(Bn, G, Hkv, M, N, K, w, n_sink, n_new, lens, data, shared):
    """Append, tables and selection by a workgroup per head in one launch against the calls one after the other: every
    output bit for bit, the padded heads of the coarse tables too."""
    wl = synth.Workload("by_head", Bn, G * Hkv, Hkv, 128, M, N, K, w, n_sink=n_sink, seed=N + K + M)
    xd = synth.make_decode_inputs(wl, device="cuda", with_kv=False)
    if data == "patterns":
        xd["codes"][:] = xd["codes"][:, :, torch.randint(0, 60, (N,), device="cuda")]
    if data == "equal":
        xd["codes"][:] = xd["codes"][:, :, :1]
    if data == "zero":
        xd["q"][0] = 0
    weights = synth.make_query_second_moment(wl)["h_diag"].cuda()
    keys = synth.make_encode_keys(wl, n_new, device="cuda", stress=True)
    dims = H.dims_of(wl)
    sel = B.make_dims(Bn, Hkv, Hkv, 128, M, N) if shared else dims
    heads = Hkv if shared else G * Hkv
    sl = None if lens is None else torch.tensor(lens, dtype=torch.int32, device="cuda")
    res = []
    for one in (False, True):
        st = B.DecodeState(dims, max(K, 1), w, n_sink, xd["q"].dtype, xd["inv_freq"], wl.wrope_b)
        lut = torch.full((B.lut_elems(sel),), -1, dtype=torch.int32, device="cuda")
        scale = torch.zeros(Bn, heads, device="cuda")
        idx = torch.full((Bn * heads * K + 8,), -7, dtype=torch.int32, device="cuda")
        score = torch.full((Bn * heads * K + 8,), -7.0, device="cuda")
        count = torch.full((Bn, heads), -7, dtype=torch.int32, device="cuda")
        codes = xd["codes"].clone()
        call = (dims, keys, n_new, N - n_new, xd["codebook"], weights, B.W_DIAG, codes, xd["q"], st.cos_b, st.sin_b, st.q_rot,
                lut, scale, K, w, n_sink, sl, idx, count, score, None)
        if one:
            (B.decode_select_shared if shared else B.decode_select)(*call)
        else:
            B.encode_keys(dims, keys, n_new, N - n_new, xd["codebook"], weights, B.W_DIAG, codes,
                          torch.empty(B.workspace_bytes(dims, B.OP_ENCODE), dtype=torch.uint8, device="cuda"))
            (B.build_lut_shared if shared else B.build_lut)(dims, xd["q"], st.cos_b, st.sin_b, xd["codebook"], st.q_rot, lut, scale)
            B.score_topk(sel, codes, lut, scale, K, w, n_sink, sl, idx, count, score, None, None)
        torch.cuda.synchronize()
        res.append((codes, lut, scale, st.q_rot, idx, count, score.view(torch.int32)))
    for i, (a, b) in enumerate(zip(*res)):
        assert torch.equal(a, b), f"output {i} differs"


@pytest.mark.parametrize("Bn,G,Hkv,M,N,K,w,n_sink,n_new,lens", [
    (40, 4, 8, 16, 16500, 400, 64, 4, 1, None),      # 320 groups, two rounds: they sample and encode
    (34, 7, 4, 32, 18000, 300, 64, 0, 2, True),      # 272, every other of three heads; ragged lengths
    (24, 4, 8, 16, 60000, 700, 64, 0, 1, None),      # 192 groups, the sample of two parts taken by one workgroup
    (24, 4, 8, 16, 70000, 700, 64, 0, 1, None),      # too many rows for one: the sampling stays a launch of its own
    (17, 4, 8, 32, 40000, 2300, 64, 4, 1, True),     # a wide selection
    (40, 4, 8, 16, 16500, 400, 64, 0, 0, None),      # nothing appended
    (24, 4, 8, 16, 17000, 400, 64, 0, 1, None),      # 192 groups, workgroups that encode wait for each other on the free CUs
    (22, 4, 8, 32, 17000, 400, 64, 0, 2, None),      # 176, too many keys for that
])
@pytest.mark.parametrize("shared", [False, True])
def test_decode_select_of_many_sequences_equals_the_calls(Bn, G, Hkv, M, N, K, w, n_sink, n_new, lens, shared):
    """Tables, sampling and append by the same workgroups, where they are more than one round of the CUs, against the calls
    one after the other, whose samples have other parts: every output bit for bit, twice in the same workspace."""
    wl = synth.Workload("many", Bn, G * Hkv, Hkv, 128, M, N, K, w, n_sink=n_sink, seed=N + K + M)
    xd = synth.make_decode_inputs(wl, device="cuda", with_kv=False)
    weights = synth.make_query_second_moment(wl)["h_diag"].cuda()
    keys = synth.make_encode_keys(wl, n_new, device="cuda", stress=True) if n_new else None
    dims = H.dims_of(wl)
    sel = B.make_dims(Bn, Hkv, Hkv, 128, M, N) if shared else dims
    heads = Hkv if shared else G * Hkv
    sl = None
    if lens:
        sl = torch.randint(0, N + 1, (Bn,), generator=torch.Generator().manual_seed(N), dtype=torch.int32).cuda()
    ws = torch.full((B.workspace_bytes(sel, B.OP_SCORE_TOPK, K, w),), 0xA5, dtype=torch.uint8, device="cuda")
    res = []
    for one in (False, True, True):
        st = B.DecodeState(dims, K, w, n_sink, xd["q"].dtype, xd["inv_freq"], wl.wrope_b)
        lut = torch.full((B.lut_elems(sel),), -1, dtype=torch.int32, device="cuda")
        scale = torch.zeros(Bn, heads, device="cuda")
        idx = torch.full((Bn * heads * K + 8,), -7, dtype=torch.int32, device="cuda")
        score = torch.full((Bn * heads * K + 8,), -7.0, device="cuda")
        count = torch.full((Bn, heads), -7, dtype=torch.int32, device="cuda")
        codes = xd["codes"].clone()
        if one:
            (B.decode_select_shared if shared else B.decode_select)(
                dims, keys, n_new, N - n_new, xd["codebook"], weights, B.W_DIAG, codes, xd["q"], st.cos_b, st.sin_b, st.q_rot,
                lut, scale, K, w, n_sink, sl, idx, count, score, ws)
        else:
            if n_new:
                B.encode_keys(dims, keys, n_new, N - n_new, xd["codebook"], weights, B.W_DIAG, codes,
                              torch.empty(B.workspace_bytes(dims, B.OP_ENCODE), dtype=torch.uint8, device="cuda"))
            (B.build_lut_shared if shared else B.build_lut)(dims, xd["q"], st.cos_b, st.sin_b, xd["codebook"], st.q_rot, lut, scale)
            B.score_topk(sel, codes, lut, scale, K, w, n_sink, sl, idx, count, score, None, ws)
        torch.cuda.synchronize()
        res.append((codes, lut, scale, st.q_rot, idx, count, score.view(torch.int32)))
    for other in res[1:]:
        for i, (a, b) in enumerate(zip(res[0], other)):
            assert torch.equal(a, b), f"output {i} differs"


@pytest.mark.parametrize("Bn,Hkv,G,M,N,K,w,n_sink,lens,rows,page", [
    (40, 2, 4, 16, 16384 + 64, 491, 64, 0, None, None, 0),               # 80 groups, the fewest candidates and groups
    (37, 4, 2, 16, 65536 + 64 + 4, 1500, 64, 4, None, None, 0),          # the most candidates of the route
    (37, 4, 2, 16, 65536 + 64 + 5, 300, 64, 4, None, None, 0),           # one more: the streaming route
    (25, 2, 7, 32, 20001, 1, 0, 17, None, None, 0),                      # two groups a KV head, the last one of three; one winner
    (90, 1, 1, 32, 17000, 2300, 64, 4, True, None, 0),                   # one head; ragged, fewer candidates than K and none
    (42, 2, 4, 16, 20000, 3700, 64, 0, None, None, 0),                   # nearly all that a list holds
    (42, 2, 3, 16, 18000, 900, 64, 4, None, "patterns", 0),              # ~450 equal scores: ties inside the band
    (42, 2, 4, 32, 18000, 900, 64, 4, None, "few", 0),                   # 6000 equal scores: lists overflow
    (43, 2, 4, 32, 17001, 700, 64, 0, True, None, 16),                   # codes in pages
])
def test_selection_by_lists_equals_a_full_sort(Bn, Hkv, G, M, N, K, w, n_sink, lens, rows, page):
    """Long contexts of many groups (one workgroup for the heads of a group, lists in LDS) against a full sort."""
    wl = synth.Workload("lists", Bn, Hkv * G, Hkv, 128, M, N, K, w, n_sink=n_sink, seed=N + K)
    xd = synth.make_decode_inputs(wl, device="cuda", with_kv=False)
    if rows:
        xd["codes"][:] = xd["codes"][:, :, torch.randint(0, 40 if rows == "patterns" else 3, (N,), device="cuda")]
    sl = None
    if lens:
        sl = torch.randint(0, N + 1, (Bn,), generator=torch.Generator().manual_seed(N), dtype=torch.int32)
        sl[:5] = torch.tensor([N, 0, w, w + n_sink + 1, min(N, w + n_sink + 1500)])
    st = B.DecodeState(H.dims_of(wl), K, w, n_sink, xd["q"].dtype, xd["inv_freq"], wl.wrope_b)
    st.topk_idx.fill_(-7), st.topk_count.fill_(-7), st.topk_score.fill_(-7.0), st.ws.fill_(0xA5)
    B.build_lut(st.dims, xd["q"], st.cos_b, st.sin_b, xd["codebook"], st.q_rot, st.lut, st.lut_scale)
    out = (st.topk_idx, st.topk_count, st.topk_score)
    dev_lens = None if sl is None else sl.cuda()
    if page:
        slots = (N + page - 1) // page
        table = torch.randperm(Bn * slots + 2, device="cuda")[:Bn * slots].reshape(Bn, slots).to(torch.int32)
        padded = torch.nn.functional.pad(xd["codes"], (0, 0, 0, slots * page - N))
        pool = torch.zeros(Bn * slots + 2, Hkv, page, M, dtype=torch.uint8, device="cuda")
        pool[table.reshape(-1).long()] = (padded.reshape(Bn, Hkv, slots, page, M).permute(0, 2, 1, 3, 4)
                                          .reshape(Bn * slots, Hkv, page, M))
        B.score_topk_paged(st.dims, pool, table, page, st.lut, st.lut_scale, K, w, n_sink, dev_lens, *out, None, st.ws)
    else:
        B.score_topk(st.dims, xd["codes"], st.lut, st.lut_scale, K, w, n_sink, dev_lens, *out, None, st.ws)
    stats = torch.empty(Bn, Hkv * G, dtype=torch.int32, device="cuda")
    B.score_topk_stats(st.dims, K, w, n_sink, st.ws, stats)
    for a, b in zip((out[0], out[1], out[2].view(torch.int32)), _full_sort(wl, xd, st, None if sl is None else sl.tolist())):
        assert torch.equal(a, b)
    if rows is None and sl is None and K <= 2048:   # no head was done again
        route = (stats.cpu().numpy().astype(np.int64) & 0xffffffff) >> 28
        assert (route == 0).all()


@pytest.mark.parametrize("Hkv,G,M,N,K,rows,page", [
    (2, 4, 16, 60000, 1500, "clumped", 0),      # the survivors of a head in two chunks: more than the LDS of a workgroup keeps
    (1, 7, 32, 100000, 2500, "clumped", 16),
    (1, 4, 16, 40000, 4000, "clumped", 0),      # ... and lists that overflow
    (1, 3, 32, (1 << 20) - 3, 2048, None, 0),   # the longest context: more candidates than leave room for the exact table
    (2, 4, 32, 65536, 1500, None, 0),           # a band of several hundred rows
    (1, 4, 16, 33000, 700, "patterns", 0),      # ~820 rows at every score
])
def test_streamed_selection_equals_a_full_sort(Hkv, G, M, N, K, rows, page):
    """The streaming route (lists of every chunk in memory) against a full sort."""
    wl = synth.Workload("stream", 1, Hkv * G, Hkv, 128, M, N, K, 64, n_sink=4, seed=N + K)
    xd = synth.make_decode_inputs(wl, device="cuda", with_kv=False)
    if rows == "patterns":
        xd["codes"][:] = xd["codes"][:, :, torch.randint(0, 40, (N,), device="cuda")]
    st = B.DecodeState(H.dims_of(wl), K, 64, 4, xd["q"].dtype, xd["inv_freq"], wl.wrope_b)
    B.build_lut(st.dims, xd["q"], st.cos_b, st.sin_b, xd["codebook"], st.q_rot, st.lut, st.lut_scale)
    if rows == "clumped":   # the best 2 K rows of the first head of every KV head come to stand together
        table = st.lut[:Hkv * G * 256 * M].view(Hkv, G, 256 * M)[:, 0].long()
        for kv in range(Hkv):
            score = table[kv][xd["codes"][0, kv].long() * M + torch.arange(M, device="cuda")].sum(1)
            order = torch.sort(score, descending=True).indices
            order = torch.cat([order[2 * K:2 * K + N // 3], order[:2 * K], order[2 * K + N // 3:]])
            xd["codes"][0, kv] = xd["codes"][0, kv][order].clone()
    st.topk_idx.fill_(-7), st.topk_count.fill_(-7), st.topk_score.fill_(-7.0), st.ws.fill_(0xA5)
    out = (st.topk_idx, st.topk_count, st.topk_score)
    if page:
        slots = (N + page - 1) // page
        table = torch.randperm(slots + 2, device="cuda")[:slots].reshape(1, slots).to(torch.int32)
        padded = torch.nn.functional.pad(xd["codes"], (0, 0, 0, slots * page - N))
        pool = torch.zeros(slots + 2, Hkv, page, M, dtype=torch.uint8, device="cuda")
        pool[table[0].long()] = padded.reshape(Hkv, slots, page, M).permute(1, 0, 2, 3).contiguous()
        B.score_topk_paged(st.dims, pool, table, page, st.lut, st.lut_scale, K, 64, 4, None, *out, None, st.ws)
    else:
        B.score_topk(st.dims, xd["codes"], st.lut, st.lut_scale, K, 64, 4, None, *out, None, st.ws)
    for a, b in zip((out[0], out[1], out[2].view(torch.int32)), _full_sort(wl, xd, st, None)):
        assert torch.equal(a, b)


def test_streamed_selections_of_several_threads_equal_a_full_sort():
    """The final kernel's LDS grows with the context: short and the longest contexts selected by threads side by side, each on
    a stream of its own."""
    def prepared(n):
        wl = synth.Workload("threads", 1, 2, 2, 128, 16, n, 500, 64, n_sink=4, seed=n)
        xd = synth.make_decode_inputs(wl, device="cuda", with_kv=False)
        st = B.DecodeState(H.dims_of(wl), 500, 64, 4, xd["q"].dtype, xd["inv_freq"], wl.wrope_b)
        B.build_lut(st.dims, xd["q"], st.cos_b, st.sin_b, xd["codebook"], st.q_rot, st.lut, st.lut_scale)
        st.topk_idx.fill_(-7), st.topk_count.fill_(-7), st.topk_score.fill_(-7.0)
        return wl, xd, st

    calls = [prepared(n) for n in (20000, 1 << 20, 33000, (1 << 20) - 70)]
    torch.cuda.synchronize()
    start = threading.Barrier(len(calls))
    failed = []

    def select(wl, xd, st):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                start.wait(timeout=60)
                for _ in range(3):
                    B.score_topk(st.dims, xd["codes"], st.lut, st.lut_scale, 500, 64, 4, None, st.topk_idx, st.topk_count,
                                 st.topk_score, None, st.ws)
                torch.cuda.current_stream().synchronize()
        except Exception as e:   # (an exception of a thread would not fail the test)
            failed.append(e)

    threads = [threading.Thread(target=select, args=c) for c in calls]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not failed
    for wl, xd, st in calls:
        for a, b in zip((st.topk_idx, st.topk_count, st.topk_score.view(torch.int32)), _full_sort(wl, xd, st, None)):
            assert torch.equal(a, b)


def _equal_rows(wl, xd, st, blocks):
    """Gives the rows of every KV head that stand at ranks first..last of its first query head's scores the code of one of them."""
    M, dev = wl.n_sub, "cuda"
    B.build_lut(st.dims, xd["q"], st.cos_b, st.sin_b, xd["codebook"], st.q_rot, st.lut, st.lut_scale)
    table = st.lut[:wl.batch * wl.n_q_heads * 256 * M].view(wl.batch, wl.n_kv_heads, wl.group, 256 * M)[:, :, 0].long()
    for b in range(wl.batch):
        for kv in range(wl.n_kv_heads):
            codes = xd["codes"][b, kv]
            score = table[b, kv][codes.long() * M + torch.arange(M, device=dev)].sum(1)
            order = torch.sort(score[wl.n_sink:wl.ctx_len - wl.window], descending=True).indices + wl.n_sink
            for first, last in blocks:
                codes[order[first:last]] = codes[order[(first + last) // 2]].clone()


# rows a head's list holds on the route of lists in LDS, and rows of about the K-th score that the final kernel of the streaming route does
LIST_ROWS, CROWD_ROWS = 5632, 8192


@pytest.mark.parametrize("Bn,Hkv,G,M,N,K,lens,blocks,route", [
    (42, 2, 4, 16, 20000, 600, None, [(100, 1123)], 0),              # 1023 equal scores, one fewer than the band holds
    (42, 2, 4, 16, 20000, 600, None, [(100, 1400)], 0),              # more than it holds
    (42, 2, 3, 32, 20000, 600, None, [(100, 4700)], 0),              # nearly all that a list holds
    (84, 1, 1, 32, 18000, 600, None, [(599, 1900)], 0),              # one of the equal rows wins
    (84, 1, 2, 16, 18000, 600, None, [(0, 600), (600, 1900)], 0),    # none of the second block
    (42, 2, 4, 16, 32768, 1000, None, [(0, 1300), (1300, 6300)], 0), # a list overflows and is made again
    (42, 2, 4, 16, 32768, 1000, None, [(0, 6300)], 2),               # and overflows again
    (42, 2, 4, 16, 20000, 1900, 1400, [], 0),                        # every candidate of short sequences wins
    (42, 2, 4, 32, 20000, 1900, 2000, [], 0),                        # nearly every one: the K-th far above a threshold of zero
    (65, 2, 3, 16, 65536 + 68, 1500, None, [(1400, 3000)], 0),       # the most candidates
    (2, 2, 4, 16, 60000, 1500, None, [(100, 1123)], 0),              # the streaming route: in its band,
    (2, 2, 4, 16, 60000, 1500, None, [(100, 8100)], 0),              # all that its final kernel ranks,
    (2, 2, 4, 16, 60000, 1500, None, [(100, 8700)], 2),              # and more
    (1, 1, 4, 32, 66000, 1500, None, [(1000, 2300)], 0),
    (1, 1, 2, 32, 1 << 20, 2048, None, [(1000, 4500)], 0),           # the longest context, whose tables stay in memory
])
def test_selection_among_equal_scores_takes_no_detour(Bn, Hkv, G, M, N, K, lens, blocks, route):
    """Many rows of the K-th score: against a full sort, and without the exact route as long as the lists hold them."""
    wl = synth.Workload("equal", Bn, Hkv * G, Hkv, 128, M, N, K, 64, n_sink=4, seed=N + K)
    xd = synth.make_decode_inputs(wl, device="cuda", with_kv=False)
    st = B.DecodeState(H.dims_of(wl), K, 64, 4, xd["q"].dtype, xd["inv_freq"], wl.wrope_b)
    lists = Bn * Hkv * ((G + 3) // 4) >= 80
    assert B.score_topk_plan(st.dims, K, 64, 4)["survivor_capacity"] == (LIST_ROWS if lists else CROWD_ROWS)
    _equal_rows(wl, xd, st, blocks)
    sl = None if lens is None else torch.full((Bn,), 64 + 4 + lens, dtype=torch.int32)
    st.topk_idx.fill_(-7), st.topk_count.fill_(-7), st.topk_score.fill_(-7.0), st.ws.fill_(0xA5)
    out = (st.topk_idx, st.topk_count, st.topk_score)
    B.score_topk(st.dims, xd["codes"], st.lut, st.lut_scale, K, 64, 4, None if sl is None else sl.cuda(), *out, None, st.ws)
    stats = torch.empty(Bn, Hkv * G, dtype=torch.int32, device="cuda")
    B.score_topk_stats(st.dims, K, 64, 4, st.ws, stats)
    for a, b in zip((out[0], out[1], out[2].view(torch.int32)), _full_sort(wl, xd, st, None if sl is None else sl.tolist())):
        assert torch.equal(a, b)
    routes = (stats.view(Bn, Hkv, G)[:, :, 0].cpu().numpy().astype(np.int64) & 0xffffffff) >> 28   # of the heads with equal scores
    assert (routes == route).all()


@pytest.mark.parametrize("call", ["score", "select"])
@pytest.mark.parametrize("M,G", [(16, 4), (32, 3)])
def test_selection_by_lists_replayed_from_a_graph(M, G, call):
    """A captured selection by lists: every replay, on new codes and queries, equals the call."""
    wl = synth.Workload("lists_graph", 42, 2 * G, 2, 128, M, 17000, 500, 64, n_sink=4, seed=M)
    xd = synth.make_decode_inputs(wl, device="cuda", with_kv=False)
    st = B.DecodeState(H.dims_of(wl), 500, 64, 4, xd["q"].dtype, xd["inv_freq"], wl.wrope_b)
    assert B.score_topk_plan(st.dims, 500, 64, 4)["survivor_capacity"] == LIST_ROWS
    key = torch.randn(42, 2, 1, 128, device="cuda")

    def run():
        if call == "select":
            B.decode_select(st.dims, key, 1, 16999, xd["codebook"], None, B.W_NONE, xd["codes"], xd["q"], st.cos_b, st.sin_b,
                            st.q_rot, st.lut, st.lut_scale, 500, 64, 4, None, st.topk_idx, st.topk_count, st.topk_score, st.ws)
        else:
            B.build_lut(st.dims, xd["q"], st.cos_b, st.sin_b, xd["codebook"], st.q_rot, st.lut, st.lut_scale)
            B.score_topk(st.dims, xd["codes"], st.lut, st.lut_scale, 500, 64, 4, None, st.topk_idx, st.topk_count, st.topk_score,
                         None, st.ws)

    run()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        run()
    for _ in range(3):
        xd["q"].copy_(torch.randn_like(xd["q"]))
        xd["codes"].copy_(xd["codes"].roll(1, 2))
        st.topk_idx.fill_(-7), st.topk_count.fill_(-7), st.topk_score.fill_(-7.0)
        graph.replay()
        got = [t.clone() for t in (st.topk_idx, st.topk_count, st.topk_score.view(torch.int32))]
        for a, b in zip(got, _full_sort(wl, xd, st, None)):
            assert torch.equal(a, b)
        run()
        for a, b in zip(got, (st.topk_idx, st.topk_count, st.topk_score.view(torch.int32))):
            assert torch.equal(a, b)


@pytest.mark.parametrize("call", ["score", "select", "paged"])
@pytest.mark.parametrize("groups,M,cand", [
    (87, 16, 24000), (87, 16, 24001), (111, 16, 28000), (111, 16, 28001), (127, 16, 32000), (127, 16, 32001), (128, 16, 36000),
    (128, 16, 36001), (95, 32, 16384), (96, 32, 18000), (111, 32, 18001), (112, 32, 26000), (127, 32, 26001), (128, 32, 36000)])
def test_selection_of_lengths_on_both_sides_of_the_line_for_lists(groups, M, cand, call):
    """Sequences of their own lengths, where the choice between the lists of a workgroup and the streaming route depends on there
    being any: either way against a full sort, by the two calls, by the one, and of codes in pages."""
    N, K, page = cand + 68, 400, 16
    wl = synth.Workload("line", groups, 1, 1, 128, M, N, K, 64, n_sink=4, seed=cand)
    xd = synth.make_decode_inputs(wl, device="cuda", with_kv=False)
    st = B.DecodeState(H.dims_of(wl), K, 64, 4, xd["q"].dtype, xd["inv_freq"], wl.wrope_b)
    sl = torch.randint(N // 4, N + 1, (groups,), generator=torch.Generator().manual_seed(N), dtype=torch.int32)
    sl[:4] = torch.tensor([N, 0, 68, 68 + K])
    st.topk_idx.fill_(-7), st.topk_count.fill_(-7), st.topk_score.fill_(-7.0), st.ws.fill_(0xA5)
    if call == "select":
        key = torch.randn(groups, 1, 1, 128, device="cuda")
        B.decode_select(st.dims, key, 1, N - 1, xd["codebook"], None, B.W_NONE, xd["codes"], xd["q"], st.cos_b, st.sin_b, st.q_rot,
                        st.lut, st.lut_scale, K, 64, 4, sl.cuda(), st.topk_idx, st.topk_count, st.topk_score, st.ws)
    else:
        B.build_lut(st.dims, xd["q"], st.cos_b, st.sin_b, xd["codebook"], st.q_rot, st.lut, st.lut_scale)
        out = (st.topk_idx, st.topk_count, st.topk_score, None, st.ws)
        if call == "paged":
            slots = (N + page - 1) // page
            table = torch.randperm(groups * slots, device="cuda").reshape(groups, slots).to(torch.int32)
            pool = torch.zeros(groups * slots, 1, page, M, dtype=torch.uint8, device="cuda")
            padded = torch.nn.functional.pad(xd["codes"], (0, 0, 0, slots * page - N))
            pool[table.reshape(-1).long()] = padded.reshape(groups * slots, 1, page, M)
            B.score_topk_paged(st.dims, pool, table, page, st.lut, st.lut_scale, K, 64, 4, sl.cuda(), *out)
        else:
            B.score_topk(st.dims, xd["codes"], st.lut, st.lut_scale, K, 64, 4, sl.cuda(), *out)
    for a, b in zip((st.topk_idx, st.topk_count, st.topk_score.view(torch.int32)), _full_sort(wl, xd, st, sl.tolist())):
        assert torch.equal(a, b)


@pytest.mark.parametrize("call", ["score", "select"])
@pytest.mark.parametrize("Bn,G,N,K,rows", [(72, 4, 8300, 200, None), (72, 4, 8300, 260, None), (72, 7, 4500, 443, None), (72, 7, 1500, 40, None),
                                           (270, 1, 8300, 800, None), (270, 1, 8300, 1200, None), (72, 4, 8300, 200, 9),
                                           (72, 4, 8300, 260, 9), (72, 4, 16384 + 68, 3000, None)])
def test_short_contexts_of_32_subspaces_by_either_kernel(Bn, G, N, K, rows, call):
    """A workgroup per group, M = 32: the kernel for bands of few rows and that for many, also where all scores are among nine,
    against a full sort."""
    wl = synth.Workload("bands", Bn, G, 1, 128, 32, N, K, 64, n_sink=4, seed=N + K)
    xd = synth.make_decode_inputs(wl, device="cuda", with_kv=False)
    if rows:
        xd["codes"][:] = xd["codes"][:, :, torch.randint(0, rows, (N,), device="cuda")]
    st = B.DecodeState(H.dims_of(wl), K, 64, 4, xd["q"].dtype, xd["inv_freq"], wl.wrope_b)
    st.topk_idx.fill_(-7), st.topk_count.fill_(-7), st.topk_score.fill_(-7.0)
    out = (st.topk_idx, st.topk_count, st.topk_score)
    if call == "select":
        key = torch.randn(Bn, 1, 1, 128, device="cuda")
        B.decode_select(st.dims, key, 1, N - 1, xd["codebook"], None, B.W_NONE, xd["codes"], xd["q"], st.cos_b, st.sin_b, st.q_rot,
                        st.lut, st.lut_scale, K, 64, 4, None, *out, st.ws)
    else:
        B.build_lut(st.dims, xd["q"], st.cos_b, st.sin_b, xd["codebook"], st.q_rot, st.lut, st.lut_scale)
        B.score_topk(st.dims, xd["codes"], st.lut, st.lut_scale, K, 64, 4, None, *out, None, st.ws)
    for a, b in zip((out[0], out[1], out[2].view(torch.int32)), _full_sort(wl, xd, st, None)):
        assert torch.equal(a, b)
