"""The work a user of this library has it do, as cases that can be timed and compared.

`listed()` names fixed cases, `draw(rng)` gives further ones of the same ranges.  Three kinds:

  step    one decode step of one layer: append the current token's key to the code matrix, rotate the
          query and build its tables, score every cached token and select the top-K, attend over the
          selected rows, the sinks and the recent window
  encode  the prefill side: codes of all keys of a batch of prompts (or of one chunk of them)
  fit     calibration: the second moment of the rotated queries, and one Lloyd iteration (assignment
          and centroids) over a set of keys

Inputs follow paper_2502_12665_amd.synth: uniform codes, keys = codeword + noise, normal queries and
values.  A code matrix of one case is up to 268 MB and its K/V cache up to 4.3 GB.
"""
from __future__ import annotations

import math

import torch

from paper_2502_12665_amd import binding as B
from paper_2502_12665_amd import synth

MAX_ROWS = 8 << 20        # cached tokens of a drawn step, over sequences and KV heads
MAX_SELECTED = 1800000    # selected rows of a drawn step, over sequences and query heads
MAX_KEYS = {16: 1800000, 32: 1800000, 1: 800000}   # keys of a drawn encode, by number of subspaces
MAX_FIT_KEYS = 1000000


def _step(name, batch, heads, kv_heads, m, ctx, top_k, window, sink=0, dtype="bf16", **opts):
    case = {"name": name, "kind": "step", "batch": batch, "heads": heads, "kv_heads": kv_heads, "m": m,
            "ctx": ctx, "top_k": top_k, "window": window, "sink": sink, "dtype": dtype,
            "shared": False, "page": 0, "ragged": False}
    case.update(opts)
    return case


def listed():
    return [
        # The smallest call: one KV head, 4096 tokens, float32 cache.  Launches and latency.
        _step("step_tiny_f32", 1, 4, 1, 16, 4096, 128, 64, dtype="f32"),
        # One interactive user: a single sequence of 32k tokens.
        _step("step_b1_32k", 1, 32, 8, 16, 32768, 1024, 128),
        # Serving many users at the context and selection ratio of the paper's throughput experiment:
        # 16k tokens, 3 % of them selected, 4 sinks and the last 64 tokens kept.
        _step("step_b64_16k", 64, 32, 8, 16, 16384, 491, 64, sink=4),
        # A few long conversations (the benchmark's default workload).
        _step("step_b4_128k", 4, 32, 8, 16, 131072, 2048, 256),
        # The paper's longest context at its selection ratio, 3 % of 96k tokens; an odd length.
        _step("step_b2_96k_3pct", 2, 32, 8, 16, 98301, 2949, 64, sink=4),
        # The largest batch: 7 query heads per KV head, 32 subspaces.
        _step("step_b32_64k_g7", 32, 28, 4, 32, 65536, 2048, 128),
        # One selection per KV head, sequences of different lengths (their codes appended elsewhere).
        _step("step_shared_ragged", 4, 32, 8, 16, 131072, 2048, 256, sink=4, shared=True, ragged=True),
        # Codes and K/V in pages of 16 tokens, as a paged serving cache holds them.
        _step("step_paged_b8_48k", 8, 32, 8, 16, 49157, 1475, 64, sink=4, page=16),
        # The paper's own quantiser: one codebook of 4096 codewords per KV head, 16-bit codes.
        _step("step_single_b4_128k", 4, 32, 8, 1, 131072, 2048, 256),
        # Prefill of four prompts of an odd length: product quantiser, per-dimension weights.
        {"name": "encode_prefill", "kind": "encode", "batch": 4, "kv_heads": 8, "m": 16, "tokens": 50001,
         "weights": "diag"},
        # Prefill of one long prompt in the paper's geometry, full weight matrix, codewords prepared once.
        {"name": "encode_single_prefill", "kind": "encode", "batch": 1, "kv_heads": 8, "m": 1, "tokens": 96001,
         "weights": "block"},
        # Calibration: query second moment and one Lloyd iteration in the paper's geometry.
        {"name": "fit_single", "kind": "fit", "batch": 4, "heads": 32, "kv_heads": 8, "m": 1, "tokens": 24001,
         "samples": 50000},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    u = rng.random()
    if u < 0.7:
        m = rng.choice([16, 16, 16, 32, 32, 1])
        heads, kv_heads = rng.choice([(32, 8), (32, 8), (28, 4), (4, 1), (16, 2)])
        ctx = _log_int(rng, 1500, 131072)
        window = rng.choice([64, 128, 256])
        # 1 % to 6 % of the context, as far as the library selects
        top_k = max(16, min(4096, int(ctx * math.exp(rng.uniform(math.log(0.01), math.log(0.06))))))
        most = min(64, MAX_ROWS // (kv_heads * ctx), MAX_SELECTED // (heads * top_k))
        batch = _log_int(rng, 1, max(1, most))
        form = rng.choice(["plain", "plain", "plain", "shared", "paged"])
        return {k: v for k, v in _step(
            "", batch, heads, kv_heads, m, ctx, top_k, window, sink=rng.choice([0, 4]),
            dtype="f32" if rng.random() < 0.15 else "bf16", shared=form == "shared" and m != 1,
            page=rng.choice([16, 64]) if form == "paged" and m != 1 else 0,
            ragged=rng.random() < 0.3).items() if k != "name"}
    if u < 0.9:
        m = rng.choice([16, 32, 1])
        kv_heads = rng.choice([1, 4, 8])
        tokens = _log_int(rng, 40, 100000)
        batch = _log_int(rng, 1, max(1, min(32, MAX_KEYS[m] // (kv_heads * tokens))))
        return {"kind": "encode", "batch": batch, "kv_heads": kv_heads, "m": m, "tokens": tokens,
                "weights": rng.choice(["none", "diag", "block"])}
    m = rng.choice([16, 32, 1])
    heads, kv_heads = rng.choice([(32, 8), (28, 4), (4, 1)])
    tokens = _log_int(rng, 2000, 60000)
    batch = _log_int(rng, 1, max(1, min(8, MAX_FIT_KEYS // (kv_heads * tokens))))
    return {"kind": "fit", "batch": batch, "heads": heads, "kv_heads": kv_heads, "m": m, "tokens": tokens,
            "samples": _log_int(rng, 2000, 50000)}


def _workload(case, seed):
    m = case["m"]
    heads = case.get("heads", case["kv_heads"])
    return synth.Workload("case", case["batch"], heads, case["kv_heads"], 128, m,
                          case.get("ctx", case.get("tokens", 0)), case.get("top_k", 0), case.get("window", 0),
                          case.get("sink", 0), kv_dtype=case.get("dtype", "bf16"), seed=seed,
                          n_centroids=4096 if m == 1 else 256)


def _dims(case, ctx, heads):
    return B.make_dims(case["batch"], heads, case["kv_heads"], 128, case["m"], ctx,
                       n_centroids=4096 if case["m"] == 1 else 256)


def _weights(wl, mode):
    """(weight_mode, weights) of a query second moment; the single codebook's block form is the full matrix."""
    hm = synth.make_query_second_moment(wl)
    if mode == "none":
        return B.W_NONE, None
    return (B.W_DIAG, hm["h_diag"].cuda()) if mode == "diag" else (B.W_BLOCK, hm["h_block"].cuda())


def _workspace(n):
    return torch.empty(max(n, 256), dtype=torch.uint8, device="cuda")


def _to_pages(x, page, table, n_pages):
    """[B, Hkv, S, W] -> pool [n_pages, Hkv, page, W] with page p of sequence b at table[b, p]."""
    b, kv, s, w = x.shape
    slots = table.shape[1]
    pool = torch.zeros(n_pages, kv, page, w, dtype=x.dtype, device=x.device)
    full = s // page
    pool[table[:, :full].reshape(-1).long()] = (x[:, :, :full * page].reshape(b, kv, full, page, w)
                                                .permute(0, 2, 1, 3, 4).reshape(b * full, kv, page, w))
    if slots > full:
        pool[table[:, full].long(), :, :s - full * page] = x[:, :, full * page:]
    return pool


def prepare(case, seed):
    return {"step": _prepare_step, "encode": _prepare_encode, "fit": _prepare_fit}[case["kind"]](case, seed)


def _prepare_step(case, seed):
    wl = _workload(case, seed)
    ctx, heads, kv_heads = case["ctx"], case["heads"], case["kv_heads"]
    x = synth.make_decode_inputs(wl, device="cuda")
    dims = _dims(case, ctx, heads)
    s = {"case": case, "dims": dims, "x": x}
    s["st"] = B.DecodeState(dims, case["top_k"], case["window"], case["sink"], x["q"].dtype, x["inv_freq"], wl.wrope_b)
    # The append: the current token's key.  A ragged batch appends through calls per sequence, which
    # are not part of this step.
    s["new_key"] = None if case["ragged"] else x["k"][:, :, ctx - 1:ctx].float().contiguous()
    s["n_new"] = 0 if case["ragged"] else 1
    s["mode"], s["weights"] = _weights(wl, "block" if case["m"] == 1 else "diag")
    s["seq_lens"] = None
    if case["ragged"]:
        g = torch.Generator().manual_seed(seed)
        lens = torch.randint(ctx // 4, ctx + 1, (case["batch"],), generator=g, dtype=torch.int32)
        lens[seed % case["batch"]] = ctx
        s["seq_lens"] = lens.cuda()
    if case["m"] == 1:
        # The encoder's workspace keeps the prepared codewords from step to step.
        s["enc_ws"] = _workspace(B.workspace_bytes(dims, B.OP_ENCODE))
        B.encode_prepare(dims, x["codebook"], s["weights"], s["mode"], s["enc_ws"])
        s["mode"] |= B.W_PREPARED
    if case["shared"]:
        s["sel_dims"] = _dims(case, ctx, kv_heads)
        dev = torch.device("cuda")
        s["lut"] = torch.empty(B.lut_elems(s["sel_dims"]), dtype=torch.int32, device=dev)
        s["lut_scale"] = torch.empty(case["batch"], kv_heads, dtype=torch.float32, device=dev)
        s["idx"] = torch.empty(case["batch"], kv_heads, case["top_k"], dtype=torch.int32, device=dev)
        s["count"] = torch.empty(case["batch"], kv_heads, dtype=torch.int32, device=dev)
        s["sel_ws"] = _workspace(B.workspace_bytes(s["sel_dims"], B.OP_SCORE_TOPK, case["top_k"], case["window"]))
    if case["page"]:
        page = case["page"]
        slots = (ctx + page - 1) // page
        n_pages = case["batch"] * slots + 3
        g = torch.Generator(device="cuda").manual_seed(seed)
        table = torch.randperm(n_pages, generator=g, device="cuda")[:case["batch"] * slots]
        table = table.reshape(case["batch"], slots).to(torch.int32)
        s["table"] = table
        for name in ("codes", "k", "v"):
            x[name] = _to_pages(x[name], page, table, n_pages)
        s["new_dims"] = _dims(case, 1, heads)
        s["new_codes"] = torch.empty(case["batch"], kv_heads, 1, case["m"], dtype=torch.uint8, device="cuda")
    return s


def _prepare_encode(case, seed):
    wl = _workload(case, seed)
    dims = _dims(case, case["tokens"], case["kv_heads"])
    s = {"case": case, "dims": dims, "codebook": synth.make_codebook(wl, "cuda"),
         "keys": synth.make_encode_keys(wl, case["tokens"], device="cuda")}
    s["mode"], s["weights"] = _weights(wl, case["weights"])
    s["ws"] = _workspace(B.workspace_bytes(dims, B.OP_ENCODE))
    s["codes"] = torch.zeros(case["batch"], case["kv_heads"], case["tokens"], case["m"], dtype=synth.code_dtype(wl),
                             device="cuda")
    if case["m"] == 1:
        B.encode_prepare(dims, s["codebook"], s["weights"], s["mode"], s["ws"])
        s["mode"] |= B.W_PREPARED
    return s


def _prepare_fit(case, seed):
    wl = _workload(case, seed)
    dims = _dims(case, case["tokens"], case["heads"])
    keys = synth.make_encode_keys(wl, case["tokens"], device="cuda")
    cb = synth.make_codebook(wl, "cuda")
    s = {"case": case, "dims": dims, "keys": keys, "codebook": cb, "new_codebook": torch.empty_like(cb)}
    g = torch.Generator(device="cuda").manual_seed(seed)
    s["queries"] = torch.randn(case["samples"], case["heads"], 128, generator=g, device="cuda", dtype=torch.float32)
    s["moment"] = torch.empty(case["kv_heads"], 128, 128, dtype=torch.float32, device="cuda")
    s["mode"], s["weights"] = _weights(wl, "block")
    s["ws"] = _workspace(max(B.workspace_bytes(dims, B.OP_ENCODE), B.workspace_bytes(dims, B.OP_FIT)))
    s["codes"] = torch.zeros(case["batch"], case["kv_heads"], case["tokens"], case["m"], dtype=synth.code_dtype(wl),
                             device="cuda")
    s["counts"] = torch.empty(case["kv_heads"], case["m"], wl.n_centroids, dtype=torch.int32, device="cuda")
    return s


def run(state):
    return {"step": _run_step, "encode": _run_encode, "fit": _run_fit}[state["case"]["kind"]](state)


def _run_step(s):
    c, dims, x, st = s["case"], s["dims"], s["x"], s["st"]
    pos0, top_k, window, sink, lens = c["ctx"] - s["n_new"], c["top_k"], c["window"], c["sink"], s["seq_lens"]
    if c["shared"]:
        B.decode_select_shared(dims, s["new_key"], s["n_new"], pos0, x["codebook"], s["weights"], s["mode"], x["codes"],
                               x["q"], st.cos_b, st.sin_b, st.q_rot, s["lut"], s["lut_scale"], top_k, window, sink, lens,
                               s["idx"], s["count"], None, s["sel_ws"])
        B.sparse_attn_shared(dims, x["q"], st.q_rot, x["k"], x["v"], s["idx"], s["count"], top_k, window, sink,
                             st.cos_win, st.sin_win, lens, st.out, st.ws)
        return {"out": st.out, "idx": s["idx"], "count": s["count"], "q_rot": st.q_rot, "codes": x["codes"]}
    if c["page"]:
        if s["n_new"]:
            B.encode_keys(s["new_dims"], s["new_key"], 1, 0, x["codebook"], s["weights"], s["mode"], s["new_codes"],
                          st.ws)
            B.codes_to_pages(dims, s["new_codes"], 1, pos0, x["codes"], s["table"], c["page"])
        B.build_lut(dims, x["q"], st.cos_b, st.sin_b, x["codebook"], st.q_rot, st.lut, st.lut_scale)
        B.score_topk_paged(dims, x["codes"], s["table"], c["page"], st.lut, st.lut_scale, top_k, window, sink, lens,
                           st.topk_idx, st.topk_count, None, None, st.ws)
        B.sparse_attn_paged(dims, x["q"], st.q_rot, x["k"], x["v"], s["table"], c["page"], st.topk_idx, st.topk_count,
                            top_k, window, sink, st.cos_win, st.sin_win, lens, st.out, st.ws)
    else:
        B.decode_select(dims, s["new_key"], s["n_new"], pos0, x["codebook"], s["weights"], s["mode"], x["codes"], x["q"],
                        st.cos_b, st.sin_b, st.q_rot, st.lut, st.lut_scale, top_k, window, sink, lens, st.topk_idx,
                        st.topk_count, None, s.get("enc_ws", st.ws))
        B.sparse_attn(dims, x["q"], st.q_rot, x["k"], x["v"], st.topk_idx, st.topk_count, top_k, window, sink,
                      st.cos_win, st.sin_win, lens, st.out, st.ws)
    return {"out": st.out, "idx": st.topk_idx, "count": st.topk_count, "q_rot": st.q_rot, "codes": x["codes"]}


def _run_encode(s):
    B.encode_keys(s["dims"], s["keys"], s["case"]["tokens"], 0, s["codebook"], s["weights"], s["mode"], s["codes"], s["ws"])
    return s["codes"]


def _run_fit(s):
    n = s["case"]["tokens"]
    B.second_moment(s["dims"], s["queries"], s["case"]["samples"], s["moment"], s["ws"])
    B.encode_keys(s["dims"], s["keys"], n, 0, s["codebook"], s["weights"], s["mode"], s["codes"], s["ws"])
    B.codebook_update(s["dims"], s["keys"], n, 0, s["codes"], s["codebook"], s["new_codebook"], s["counts"], s["ws"])
    return {"moment": s["moment"], "codes": s["codes"], "codebook": s["new_codebook"], "counts": s["counts"]}


def work(case):
    m, batch, kv_heads = case["m"], case["batch"], case["kv_heads"]
    code_bytes = 2 if m == 1 else m                      # per cached token and KV head
    centroids = 4096 if m == 1 else 256                  # per subspace
    codebook = kv_heads * centroids * 128 * 4.0
    if case["kind"] == "step":
        heads, ctx, window, sink = case["heads"], case["ctx"], case["window"], case["sink"]
        rows = 0.0                                       # cached tokens, over the batch
        if case["ragged"]:
            rows = (batch - 1) * ctx * 0.625 + ctx
        else:
            rows = float(batch * ctx)
        selectors = kv_heads if case["shared"] else heads
        top_k = min(case["top_k"], max(ctx - window - sink, 0))
        row = 2 * 128 * (4 if case["dtype"] == "f32" else 2)
        kept = batch * kv_heads * (window + sink)
        attended = batch * heads * (top_k + window + sink)
        return {"bytes": rows * kv_heads * code_bytes + codebook + batch * selectors * top_k * (row + 4.0) + kept * row
                + batch * heads * 128 * 12.0,
                "flops": rows * selectors * m + batch * heads * centroids * 128 * 2.0 + attended * 128 * 4.0}
    keys = float(batch * kv_heads * case["tokens"])
    encode = {"bytes": keys * (512 + code_bytes) + codebook,
              "flops": keys * centroids * 128 * 2 + (keys * 128 * 128 * 2 if m == 1 else 0)}
    if case["kind"] == "encode":
        return encode
    queries = float(case["samples"] * case["heads"])
    return {"bytes": encode["bytes"] + keys * (512 + code_bytes) + 2 * codebook + queries * 512,
            "flops": encode["flops"] + keys * 128 + queries * 128 * 128}


def tolerance(case):
    if case["kind"] == "encode":
        return "exact"                                   # codes are the argmin of float64 distortions
    if case["kind"] == "fit":
        return {"rel": 2e-7, "max": 1e-6}                # float64 sums, rounded once to float32
    # Selections are exact.  The attention sums in float32: against float64 a float32 output is off by
    # 1.6e-7, a bfloat16 one by up to 6e-5 (a few values round the other way; more where few are large).
    return {"rel": 2e-6} if case["dtype"] == "f32" else {"rel": 1e-3}
