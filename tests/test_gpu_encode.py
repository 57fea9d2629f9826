"""The product-quantiser encoder against the float64 argmin of the definition, at the sizes and values where its
matrix-core filter could go wrong."""
import pytest
import torch

from paper_2502_12665_amd import binding as B
from paper_2502_12665_amd import synth

pytestmark = pytest.mark.gpu


def _distortions(keys, codebook, weights, mode):
    """float64 (k - c) H (k - c)^T of every key, subspace and centroid: [B, Hkv, n, M, 256]."""
    kv, m, _, ds = codebook.shape
    k = keys.double().reshape(*keys.shape[:3], m, 1, ds)
    e = k - codebook.double()[None, :, None]
    if mode == B.W_DIAG:
        return (e * e * weights.double().reshape(kv, m, ds)[None, :, None, :, None]).sum(-1)
    if mode == B.W_BLOCK:
        out = torch.empty(e.shape[:-1], dtype=torch.float64, device=keys.device)
        for h in range(kv):
            for s in range(m):
                x = e[:, h, :, s].contiguous()
                out[:, h, :, s] = ((x @ weights[h, s].double()) * x).sum(-1)
        return out
    return (e * e).sum(-1)


def _encode(dims, keys, codebook, weights, mode, stride, m, offset=0):
    flat = torch.full((keys.shape[0] * keys.shape[1] * stride * m + 8,), 0xEE, dtype=torch.uint8, device="cuda")
    ws = torch.empty(max(B.workspace_bytes(dims, B.OP_ENCODE), 16), dtype=torch.uint8, device="cuda")
    codes = flat[offset:offset + flat.numel() - 8].view(keys.shape[0], keys.shape[1], stride, m)
    B.encode_keys(dims, keys, keys.shape[2], 3, codebook, weights, mode, codes, ws)
    torch.cuda.synchronize()
    assert (flat[:offset] == 0xEE).all() and (flat[flat.numel() - 8 + offset:] == 0xEE).all()
    assert (codes[:, :, :3] == 0xEE).all() and (codes[:, :, 3 + keys.shape[2]:] == 0xEE).all()
    return codes[:, :, 3:3 + keys.shape[2]].long()


@pytest.mark.parametrize("m,mode", [(16, "none"), (16, "diag"), (16, "block"), (32, "none"), (32, "diag"), (32, "block")])
@pytest.mark.parametrize("n_new,batch,kv", [(33, 1, 1), (64, 2, 3), (65, 1, 2), (1024, 1, 1), (1087, 2, 1), (5000, 1, 2)])
def test_codes_are_the_float64_argmin(m, mode, n_new, batch, kv):
    wl = synth.Workload("enc", batch, kv, kv, 128, m, n_new + 8, 16, 16, seed=n_new + m)
    hm = synth.make_query_second_moment(wl)
    code = {"none": B.W_NONE, "diag": B.W_DIAG, "block": B.W_BLOCK}[mode]
    weights = {"none": None, "diag": hm["h_diag"].cuda(), "block": hm["h_block"].cuda()}[mode]
    codebook = synth.make_codebook(wl, "cuda")
    ds = 128 // m
    dims = B.make_dims(batch, kv, kv, 128, m, n_new + 8)
    keys = synth.make_encode_keys(wl, n_new, device="cuda", stress=n_new % 2 == 0)
    keys[:, :, 5] *= 40.0                                     # far outside the codebook
    keys[:, :, 6] *= 1e4
    keys[:, :, 7] = 0.0
    keys[:, :, 8] *= 1e-6
    midpoint = 0.5 * (codebook[:, :, 17] + codebook[:, :, 201]).reshape(kv, 128)
    keys[:, :, 9] = midpoint                                  # two centroids about equally far
    for scale in (1.0, 3e-9, 1e12):                           # (a power of two apart or not, small or large)
        cb, ks = codebook * scale, keys * scale
        got = _encode(dims, ks, cb, weights, code, n_new + 8, m)
        dist = _distortions(ks, cb, weights, code)
        best = dist.min(-1).values
        mine = dist.gather(-1, got[..., None])[..., 0]
        # the definition's own float64 rounding, relative to the terms that cancel in k - c
        norm = ks.double().reshape(*ks.shape[:3], m, ds).pow(2).sum(-1) + cb.double().pow(2).sum(-1).amax(-1)[None, :, None]
        wmax = 1.0 if weights is None else float(weights.abs().max()) * ds
        assert ((mine - best) <= 1e-13 * wmax * norm).all(), float(((mine - best) / norm).max())


@pytest.mark.parametrize("m", [16, 32])
def test_ties_go_to_the_lower_code_and_values_that_are_not_finite_to_code_0(m):
    ds, n = 128 // m, 200
    wl = synth.Workload("enc_ties", 1, 1, 1, 128, m, n + 8, 16, 16, seed=m)
    codebook = synth.make_codebook(wl, "cuda")
    codebook[:, :, 128:] = codebook[:, :, :128]               # every centroid twice
    keys = synth.make_encode_keys(wl, n, device="cuda")
    keys[0, 0, 10] = float("nan")
    keys[0, 0, 11] = float("inf")
    dims = B.make_dims(1, 1, 1, 128, m, n + 8)
    for offset in (0, 1):                                     # (codes may start at any byte)
        got = _encode(dims, keys, codebook, None, B.W_NONE, n + 8, m, offset)
        assert (got < 128).all()
        assert (got[0, 0, 10:12] == 0).all()
        dist = _distortions(keys, codebook, None, B.W_NONE)
        ok = torch.ones(n, dtype=torch.bool, device="cuda")
        ok[10:12] = False
        first = (dist == dist.min(-1, keepdim=True).values).int().argmax(-1)
        assert torch.equal(got[0, 0][ok], first[0, 0][ok])
    broken = codebook.clone()
    broken[0, 3, 5] = float("nan")                            # a centroid that is never the nearest
    broken[0, 4] = 0.0                                        # a subspace that cannot tell its centroids apart
    keys[0, 0, 10:12] = 0.0
    got = _encode(dims, keys, broken, None, B.W_NONE, n + 8, m)
    dist = _distortions(keys, broken, None, B.W_NONE).nan_to_num(nan=float("inf"))
    first = (dist == dist.min(-1, keepdim=True).values).int().argmax(-1)
    assert torch.equal(got, first)


def _single(dims, keys, codebook, weights, mode, stride, prepared=False):
    codes = torch.full((keys.shape[0], keys.shape[1], stride), -2, dtype=torch.int16, device="cuda")
    ws = torch.empty(B.workspace_bytes(dims, B.OP_ENCODE), dtype=torch.uint8, device="cuda").fill_(0xA5)
    if prepared:
        B.encode_prepare(dims, codebook, weights, mode, ws)
        mode |= B.W_PREPARED
    B.encode_keys(dims, keys, keys.shape[2], 3, codebook, weights, mode, codes, ws)
    torch.cuda.synchronize()
    assert (codes[:, :, :3] == -2).all() and (codes[:, :, 3 + keys.shape[2]:] == -2).all()
    return codes[:, :, 3:3 + keys.shape[2]].long()


@pytest.mark.parametrize("mode", ["none", "diag", "block"])
@pytest.mark.parametrize("n_new,batch,kv", [(9, 1, 1), (129, 2, 3), (1025, 1, 8), (8200, 2, 4), (66000, 2, 2)])
def test_single_codebook_codes_are_the_float64_argmin(mode, n_new, batch, kv):
    """Short calls, and the f16 filter's (odd sizes) and the i8 filter's 32 and 128 keys per wave; keys drawn like the codewords
    leave some open.  (Both filters at each width: test_single_codebook_products.)"""
    wl = synth.Workload("enc1", batch, kv, kv, 128, 1, n_new + 8, 16, 16, seed=n_new, n_centroids=4096)
    hm = synth.make_query_second_moment(wl)
    code = {"none": B.W_NONE, "diag": B.W_DIAG, "block": B.W_BLOCK}[mode]
    weights = {"none": None, "diag": hm["h_diag"].cuda(), "block": hm["h_block"].cuda()}[mode]
    codebook = synth.make_codebook(wl, "cuda")
    dims = B.make_dims(batch, kv, kv, 128, 1, n_new + 8, n_centroids=4096)
    keys = synth.make_encode_keys(wl, n_new, device="cuda", stress=n_new % 2 == 1)
    keys[:, :, 2] *= 1e5                                      # beyond f16
    keys[:, :, 3] = 0.0
    keys[:, :, 4] *= 1e-6
    keys[:, :, 5] = 0.5 * (codebook[:, 0, 17] + codebook[:, 0, 2001])
    h64 = {"none": torch.eye(128, dtype=torch.float64, device="cuda").expand(kv, 128, 128)}.get(mode)
    if h64 is None:
        h64 = torch.diag_embed(weights.double()) if mode == "diag" else weights.double().reshape(kv, 128, 128)
    for scale in (1.0, 3e-7):
        cb, ks = codebook * scale, keys * scale
        got = _single(dims, ks, cb, weights, code, n_new + 8, prepared=scale == 1.0)
        for h in range(kv):
            c = cb[h, 0].double()
            w = c @ h64[h]
            half = 0.5 * (w * c).sum(-1)
            for b in range(batch):
                k = ks[b, h].double()
                score = half - k @ w.t()
                lost = score.gather(1, got[b, h][:, None])[:, 0] - score.min(1).values
                norm = half.max() + k.norm(dim=1) * w.norm(dim=1).max()
                assert (lost <= 1e-13 * norm).all(), float((lost / norm).max())


@pytest.mark.parametrize("mode", ["none", "block"])
@pytest.mark.parametrize("n_new,batch,kv", [(10, 1, 1), (97, 2, 3), (13001, 1, 8), (25700, 1, 8)])
def test_single_codebook_keys_near_their_codewords(n_new, batch, kv, mode):
    """Short calls and the i8 filter's 64 and 128 keys a wave, whose last tiles are ragged; some keys halfway between two
    codewords of one group of four, of one lane and of two, far out, and not finite."""
    wl = synth.Workload("enc1_near", batch, kv, kv, 128, 1, n_new + 8, 16, 16, seed=n_new, n_centroids=4096)
    weights, h64 = None, torch.eye(128, dtype=torch.float64, device="cuda").expand(kv, 128, 128)
    if mode == "block":
        weights = synth.make_query_second_moment(wl)["h_block"].cuda()
        h64 = weights.double().reshape(kv, 128, 128)
    codebook = synth.make_codebook(wl, "cuda")
    keys = synth.make_encode_keys(wl, n_new, device="cuda")
    for at, (c, d) in enumerate([(40, 42), (1000, 1016), (3, 4095)]):
        keys[:, :, n_new - 1 - at] = 0.5 * (codebook[:, 0, c] + codebook[:, 0, d])
    keys[:, :, 1] *= 300.0
    keys[:, 0, 2], keys[:, 0, 3] = float("nan"), float("inf")
    dims = B.make_dims(batch, kv, kv, 128, 1, n_new + 8, n_centroids=4096)
    got = _single(dims, keys, codebook, weights, B.W_NONE if mode == "none" else B.W_BLOCK, n_new + 8)
    assert (got[:, 0, 2:4] == 0).all()
    keys[:, 0, 2:4] = 0.0
    for h in range(kv):
        c = codebook[h, 0].double()
        w = c @ h64[h]
        half = 0.5 * (w * c).sum(-1)
        for b in range(batch):
            k = keys[b, h].double()
            score = half - k @ w.t()
            lost = score.gather(1, got[b, h][:, None])[:, 0] - score.min(1).values
            if h == 0:
                lost[2:4] = 0.0
            # (float64 sums of 128 products, of L L^T instead of H)
            assert (lost <= 1e-13 * (half.max() + k.norm(dim=1) * w.norm(dim=1).max())).all(), float(lost.max())


def _prepared_at(kv, region):
    """Where a region of the encoder's workspace begins, as enc_single_ws lays them out."""
    per_head = [128 * 128 * 8, 128 * 8, 128 * 128 * 8, 16 * 128 * 8, 4 * 128 * 4, 128 * 4096 * 8, 128 * 4096 * 8, 4096 * 8,
                4096 * 512, 4096 * 4, 4096 * 256, 4096 * 4, 4096 * 128, 4096 * 4, 128, 32 * 128 * 8, 128 * 8]
    return sum((kv * n + 255) // 256 * 256 for n in per_head[:region])


def _chosen_filters(ws, kv):
    """What a call left in its workspace: per KV head 1 if its sample took the i8 filter and 0 if the f16 one, and neither where
    there was no filter."""
    at = _prepared_at(kv, 17)
    return ws[at:at + 4 * kv].view(torch.int32).tolist()


@pytest.mark.parametrize("mode", ["none", "block"])
@pytest.mark.parametrize("n_new,batch,kv,kinds,products", [
    (9, 1, 1, "near", "sample"), (9, 1, 2, "mixed", "sample"), (128, 1, 3, "mixed", "sample"), (43, 3, 2, "mixed", "sample"),
    (3072, 1, 2, "mixed", "sample"), (257, 3, 5, "mixed", "sample"),
    (3073, 1, 1, "near", "chosen"), (777, 1, 8, "near", "chosen"), (777, 1, 8, "mixed", "chosen"), (401, 3, 8, "mixed", "chosen"),
    (13001, 1, 8, "mixed", "chosen"), (13001, 1, 8, "normal", "chosen"), (6501, 2, 8, "near", "chosen"),
    (25700, 1, 8, "mixed", "chosen"), (25700, 1, 8, "normal", "chosen"),
    (9, 1, 25, "mixed", "f16"), (799, 1, 25, "near", "f16"), (801, 1, 25, "mixed", "chosen"),
])
def test_single_codebook_products(n_new, batch, kv, kinds, products, mode):
    """Which products see the keys first, for keys near their codewords, keys drawn like the codewords and calls with KV heads of
    both: the edges of the choice, 32, 64 and 128 keys a wave with ragged tiles, of both filters.  Some keys, not among the
    sampled ones, are halfway between two codewords, far out, or not finite."""
    wl = synth.Workload("enc1_products", batch, kv, kv, 128, 1, n_new + 8, 16, 16, seed=n_new + kv, n_centroids=4096)
    weights, h64 = None, torch.eye(128, dtype=torch.float64, device="cuda").expand(kv, 128, 128)
    if mode == "block":
        weights = synth.make_query_second_moment(wl)["h_block"].cuda()
        h64 = weights.double().reshape(kv, 128, 128)
    codebook = synth.make_codebook(wl, "cuda")
    keys = synth.make_encode_keys(wl, n_new, device="cuda")
    normal = [kinds == "normal" or (kinds == "mixed" and h % 2 == 1) for h in range(kv)]
    keys[:, normal] = synth.make_encode_keys(wl, n_new, device="cuda", stress=True)[:, normal]
    rows = batch * n_new
    sampled = {(2 * at + 1) * rows // 256 for at in range(128)}
    free = [r for r in range(rows) if r not in sampled] if rows > 256 else list(range(rows))
    spots = [(r // n_new, r % n_new) for r in free[:4] + free[-4:]]
    for (b, j), (c, d) in zip(spots, [(40, 42), (1000, 1016), (3, 4095), (7, 8)]):
        keys[b, :, j] = 0.5 * (codebook[:, 0, c] + codebook[:, 0, d])
    keys[spots[4][0], :, spots[4][1]] *= 300.0
    keys[spots[5][0], :, spots[5][1]] = 0.0
    broken = spots[6:]
    for (b, j), value in zip(broken, ("nan", "inf")):
        keys[b, :, j, 5] = float(value)
    dims = B.make_dims(batch, kv, kv, 128, 1, n_new + 8, n_centroids=4096)
    ws = torch.full((B.workspace_bytes(dims, B.OP_ENCODE),), 0xA5, dtype=torch.uint8, device="cuda")
    codes = torch.full((batch, kv, n_new + 8), -2, dtype=torch.int16, device="cuda")
    B.encode_keys(dims, keys, n_new, 3, codebook, weights, B.W_NONE if mode == "none" else B.W_BLOCK, codes, ws)
    torch.cuda.synchronize()
    assert (codes[:, :, :3] == -2).all() and (codes[:, :, 3 + n_new:] == -2).all()
    got = codes[:, :, 3:3 + n_new].long()
    filters = _chosen_filters(ws, kv)
    if products == "sample":
        assert all(f not in (0, 1) for f in filters)
    else:
        assert filters == [1 if products == "chosen" and not x else 0 for x in normal]
    for b, j in broken:
        assert (got[b, :, j] == 0).all()
        keys[b, :, j] = 0.0
    for h in range(kv):
        c = codebook[h, 0].double()
        w = c @ h64[h]
        half = 0.5 * (w * c).sum(-1)
        for b in range(batch):
            k = keys[b, h].double()
            score = half - k @ w.t()
            lost = score.gather(1, got[b, h][:, None])[:, 0] - score.min(1).values
            for at, j in broken:
                if at == b:
                    lost[j] = 0.0
            # (float64 sums of 128 products, of L L^T instead of H)
            assert (lost <= 1e-13 * (half.max() + k.norm(dim=1) * w.norm(dim=1).max())).all(), float(lost.max())


def test_single_codebook_ties_and_values_that_are_not_finite():
    n = 700
    wl = synth.Workload("enc1_ties", 1, 2, 2, 128, 1, n + 8, 16, 16, seed=5, n_centroids=4096)
    codebook = synth.make_codebook(wl, "cuda")
    codebook[:, :, 2048:] = codebook[:, :, :2048]             # every codeword twice: float64 decides every key
    keys = synth.make_encode_keys(wl, n, device="cuda")
    keys[0, 1, 10], keys[0, 1, 11] = float("nan"), float("inf")
    dims = B.make_dims(1, 2, 2, 128, 1, n + 8, n_centroids=4096)
    got = _single(dims, keys, codebook, None, B.W_NONE, n + 8)
    want = synth.make_encode_keys(wl, n, device="cuda")
    for h in range(2):
        score = 0.5 * codebook[h, 0].double().pow(2).sum(-1) - want[0, h].double() @ codebook[h, 0].double().t()
        first = score[:, :2048].argmin(1)
        ok = torch.ones(n, dtype=torch.bool, device="cuda")
        if h == 1:
            ok[10:12] = False
            assert (got[0, 1, 10:12] == 0).all()
        assert torch.equal(got[0, h][ok], first[ok])


@pytest.mark.parametrize("mode", ["none", "block"])
def test_single_codebook_keys_short_against_codewords_of_one_length(mode):
    """Scores 1/2 |c^z|^2 - k . w whose first term is common to all codewords up to its last bits: the rounding of the
    sums is relative to that term, not to |k| |w|, and the second term alone decides."""
    kv, n = 2, 2000
    wl = synth.Workload("enc1_short", 1, kv, kv, 128, 1, n + 8, 16, 16, seed=11, n_centroids=4096)
    h64 = torch.eye(128, dtype=torch.float64, device="cuda").expand(kv, 128, 128)
    weights = None
    if mode == "block":
        weights = synth.make_query_second_moment(wl)["h_block"].cuda().reshape(kv, 128, 128).contiguous()
        h64 = weights.double()
    codebook = synth.make_codebook(wl, "cuda")
    z = codebook.double() @ torch.linalg.cholesky(h64)[:, None]
    codebook = (codebook / z.norm(dim=-1, keepdim=True)).float().contiguous()
    dims = B.make_dims(1, kv, kv, 128, 1, n + 8, n_centroids=4096)
    unit = synth.make_encode_keys(wl, n, device="cuda", stress=True)
    unit = unit / unit.norm(dim=-1, keepdim=True)
    for size in (1e-1, 1e-2, 1e-3, 1e-4, 1e-5, 1e-6):
        keys = (unit * size).contiguous()
        got = _single(dims, keys, codebook, weights, B.W_NONE if mode == "none" else B.W_BLOCK, n + 8)
        for h in range(kv):
            c, k = codebook[h, 0].double(), keys[0, h].double()
            w = c @ h64[h]
            half = 0.5 * (w * c).sum(-1)
            score = half - k @ w.t()
            lost = score.gather(1, got[0, h][:, None])[:, 0] - score.min(1).values
            # (float64 sums of 128 products, of L L^T instead of H)
            assert (lost <= 1e-13 * (half.max() + k.norm(dim=1) * w.norm(dim=1).max())).all(), (size, int((lost > 1e-13).sum()))


@pytest.mark.parametrize("rank", [1, 5])
@pytest.mark.parametrize("n", [20, 3001])
def test_single_codebook_weights_without_full_rank(rank, n):
    """H of few queries: rounded to float32 it has small negative eigenvalues, and so c H c^T of some codewords (the first 64,
    orthogonal to the queries).  The bound on |c H c^T| is that of the magnitudes, and codes still minimise the distortion."""
    kv = 2
    wl = synth.Workload("enc1_rank", 1, kv, kv, 128, 1, n + 8, 16, 16, seed=n + rank, n_centroids=4096)
    codebook = synth.make_codebook(wl, "cuda")
    g = torch.Generator(device="cuda").manual_seed(rank)
    basis = torch.linalg.qr(torch.randn(kv, 128, rank, generator=g, device="cuda", dtype=torch.float64)).Q
    weights = (128.0 * basis @ basis.transpose(1, 2).contiguous()).float()
    weights = torch.tril(weights) + torch.tril(weights, -1).transpose(1, 2)
    flat = codebook[:, 0, :64].double()
    codebook[:, 0, :64] = (flat - (flat @ basis) @ basis.transpose(1, 2).contiguous()).float()
    codebook = torch.stack([codebook[:, :, :2048], -codebook[:, :, :2048]], 3).reshape(codebook.shape).contiguous()   # no centre
    keys = synth.make_encode_keys(wl, n, device="cuda", stress=True)
    dims = B.make_dims(1, kv, kv, 128, 1, n + 8, n_centroids=4096)
    ws = torch.full((B.workspace_bytes(dims, B.OP_ENCODE),), 0xA5, dtype=torch.uint8, device="cuda")
    codes = torch.full((1, kv, n + 8), -2, dtype=torch.int16, device="cuda")
    B.encode_keys(dims, keys, n, 0, codebook, weights.contiguous(), B.W_BLOCK, codes, ws)
    most = ws[_prepared_at(kv, 14):][:kv * 128].view(torch.float32).view(kv, 32)[:, 2]
    for h in range(kv):
        c, k, got = codebook[h, 0].double(), keys[0, h].double(), codes[0, h, :n].long()
        w = c @ weights[h].double()
        half = 0.5 * (w * c).sum(-1)
        assert half.min() < 0.0
        assert 0.999 * half.abs().max() <= most[h] <= 1.001 * half.abs().max()
        score = half - k @ w.t()
        lost = score.gather(1, got[:, None])[:, 0] - score.min(1).values
        assert (lost <= 1e-13 * (half.max() + k.norm(dim=1) * w.norm(dim=1).max())).all(), float(lost.max())


@pytest.mark.parametrize("mode", ["none", "diag", "block"])
@pytest.mark.parametrize("n", [12, 3001])
@pytest.mark.parametrize("close", [2, 3, 40])
def test_single_codebook_keys_far_out_among_codewords_close_to_them(close, n, mode):
    """Several codewords around a long key, at distances that differ by far less than float64 rounds |k| |w|: long in the first 64
    dimensions, where they are all alike, and told apart in the others.  Every code is the argmin of the distances themselves."""
    kv, spots = 2, 9
    g = torch.Generator(device="cuda").manual_seed(close * 100000 + n)
    randn = lambda *shape: torch.randn(*shape, generator=g, device="cuda", dtype=torch.float64)
    codebook = (randn(kv, 1, 4096, 128) * torch.where(torch.arange(128, device="cuda") < 64, 100.0, 1e-3)).float()
    keys = torch.empty(1, kv, n, 128, device="cuda")
    for h in range(kv):
        at = torch.randperm(4096, generator=g, device="cuda")[:spots * close].view(spots, close)
        codebook[h, 0, at.view(-1), :64] = codebook[h, 0, at[:, :1].expand(-1, close).reshape(-1), :64]
        # distances of 1e-6 to 2e-6
        near = codebook[h, 0, at[:, 0], 64:].double()[torch.arange(n, device="cuda") % spots]
        keys[0, h, :, :64] = codebook[h, 0, at[:, 0], :64][torch.arange(n, device="cuda") % spots]
        keys[0, h, :, 64:] = (near + 1e-9 * randn(n, 64)).float()
        step = randn(spots, close, 64)
        step *= 1e-6 * (1.0 + torch.rand(spots, close, 1, generator=g, device="cuda", dtype=torch.float64)) / step.norm(dim=-1, keepdim=True)
        codebook[h, 0, at, 64:] = (codebook[h, 0, at[:, :1], 64:].double() + step).float()
    half = randn(kv, 128, 128)
    h64 = {"none": torch.eye(128, device="cuda", dtype=torch.float64).expand(kv, 128, 128),
           "diag": torch.diag_embed(half[:, 0].abs() + 0.1),
           "block": half @ half.transpose(1, 2).contiguous() / 128.0 + torch.eye(128, device="cuda", dtype=torch.float64)}[mode]
    h32 = h64.float()
    weights = {"none": None, "diag": torch.diagonal(h32, dim1=1, dim2=2).contiguous(), "block": h32.contiguous()}[mode]
    dims = B.make_dims(1, kv, kv, 128, 1, n + 8, n_centroids=4096)
    got = _single(dims, keys, codebook, weights, {"none": B.W_NONE, "diag": B.W_DIAG, "block": B.W_BLOCK}[mode], n + 8)
    for h in range(kv):
        low = torch.tril(h32[h]).double()
        sym = low + torch.tril(low, -1).t().contiguous()
        for j0 in range(0, n, 64):
            e = keys[0, h, j0:j0 + 64, None].double() - codebook[h, 0].double()
            dist = ((e @ sym) * e).sum(-1)
            lost = dist.gather(1, got[0, h, j0:j0 + 64, None])[:, 0] - dist.min(1).values
            # (w is rounded in 64 bits, 128 products of |H| |c| each, and meets sums of two distances; what the
            # distances differ by is of the order of their squares, 1e-12)
            bound = 128 * 2.0 ** -53 * float(sym.norm()) * 2000.0 * 4e-6
            assert bound < 1e-14 and (lost <= bound).all(), (float(lost.max()), bound)


@pytest.mark.parametrize("kv,n", [(8, 12001), (8, 20100), (2, 33000)])
def test_single_codebook_long_lists_of_undecided_keys(kv, n):
    """Every codeword twice, so the filter decides no key: lists of 24 to 129 chunks of 256 keys per KV head, by 64 (of 8
    heads) or 256 (of 2) workgroups each: in slices of the codewords, and with a second chunk for some workgroups."""
    wl = synth.Workload("enc1_lists", 1, kv, kv, 128, 1, n + 8, 16, 16, seed=n, n_centroids=4096)
    codebook = synth.make_codebook(wl, "cuda")
    codebook[:, :, 2048:] = codebook[:, :, :2048]
    keys = synth.make_encode_keys(wl, n, device="cuda", stress=True)
    dims = B.make_dims(1, kv, kv, 128, 1, n + 8, n_centroids=4096)
    got = _single(dims, keys, codebook, None, B.W_NONE, n + 8)
    for h in range(kv):
        c = codebook[h, 0, :2048].double()
        assert torch.equal(got[0, h], (0.5 * c.pow(2).sum(-1) - keys[0, h].double() @ c.t()).argmin(1))


@pytest.mark.parametrize("m", [16, 32])
@pytest.mark.parametrize("smallest", [1e-2, 1e-4, 1e-6])
def test_codes_under_blocks_that_are_far_from_round(m, smallest):
    """Keys about midway between two centroids, all far out along the direction that a block of H weighs least: z = k L is
    short, but its rounding is that of |k| |L|."""
    ds, n = 128 // m, 20000
    g = torch.Generator(device="cuda").manual_seed(m)
    rand = lambda *shape: torch.randn(*shape, generator=g, device="cuda", dtype=torch.float64)
    basis = torch.linalg.qr(rand(m, ds, ds)).Q
    weigh = torch.ones(ds, dtype=torch.float64, device="cuda")
    weigh[0] = smallest
    weights = (basis * weigh @ basis.transpose(-1, -2)).float()
    weights = (0.5 * (weights + weights.transpose(-1, -2))).contiguous()
    back = torch.linalg.inv(torch.linalg.cholesky(weights.double()))
    # in z: clusters of four centroids (consecutive ones, and ones far apart in the codebook)
    z = (4.0 * rand(m, 64, 1, ds) + 0.7 * rand(m, 64, 4, ds)).reshape(m, 256, ds)
    z[:, 128:] = z[:, 128:].reshape(m, 32, 4, ds).transpose(1, 2).reshape(m, 128, ds)
    codebook = (z @ back).float()[None].contiguous()
    dims = B.make_dims(1, 1, 1, 128, m, n + 8)
    at = torch.randint(0, 256, (n,), generator=g, device="cuda")
    cluster, member = torch.where(at < 128, at // 4, at % 32), torch.where(at < 128, at % 4, (at - 128) // 32)
    other = torch.where(at < 128, cluster * 4 + (member + 1) % 4, 128 + cluster + 32 * ((member + 1) % 4))
    keys = 0.5 * (codebook[0][:, at].double() + codebook[0][:, other].double()) + 1e-4 * rand(m, n, ds) @ back
    keys = keys.float().permute(1, 0, 2).reshape(1, 1, n, 128).contiguous()
    got = _encode(dims, keys, codebook, weights[None].contiguous(), B.W_BLOCK, n + 8, m)
    wrong = 0
    for first in range(0, n, 5000):
        part = keys[:, :, first:first + 5000]
        dist = _distortions(part, codebook, weights[None], B.W_BLOCK)
        best = dist.min(-1).values
        mine = dist.gather(-1, got[:, :, first:first + 5000, :, None])[..., 0]
        # (the definition's own rounding: terms of |k - c|^2)
        far = (part.double().reshape(1, 1, -1, m, ds) - codebook[0].double()[torch.arange(m, device="cuda"), got[:, :, first:first + 5000]]).pow(2).sum(-1)
        wrong += int((mine - best > 1e-13 * ds * far).sum())
    assert wrong == 0


@pytest.mark.parametrize("mode", ["none", "diag", "block"])
@pytest.mark.parametrize("n_new,data", [(8, "shifted"), (3000, "shifted"), (3000, "uneven"), (3000, "outliers")])
def test_single_codebook_away_from_the_origin_and_under_uneven_weights(mode, n_new, data):
    """Keys and codewords with much in common, weights over six orders of magnitude, and a few codewords far out, infinite or
    not a number among many, which must not move the centre that all are taken relative to."""
    kv = 2
    wl = synth.Workload("enc1_shift", 1, kv, kv, 128, 1, n_new + 8, 16, 16, seed=n_new + len(data), n_centroids=4096)
    g = torch.Generator(device="cuda").manual_seed(5)
    h64 = synth.make_query_second_moment(wl)["H"].cuda()
    if data == "uneven":
        scale = torch.logspace(-1.5, 1.5, 128, dtype=torch.float64, device="cuda")[torch.randperm(128, generator=g, device="cuda")]
        h64 = scale[:, None] * h64 * scale[None, :]
    weights, code = {"none": (None, B.W_NONE), "diag": (torch.diagonal(h64, dim1=1, dim2=2).float().contiguous(), B.W_DIAG),
                     "block": (h64.float().contiguous(), B.W_BLOCK)}[mode]
    h64 = {"none": lambda: torch.eye(128, dtype=torch.float64, device="cuda").expand(kv, 128, 128),
           "diag": lambda: torch.diag_embed(weights.double()), "block": lambda: weights.double()}[mode]()
    h64 = 0.5 * (h64 + h64.transpose(1, 2))
    codebook = synth.make_codebook(wl, "cuda")
    keys = synth.make_encode_keys(wl, n_new, device="cuda", stress=True)
    if data == "shifted":
        shift = 40.0 * torch.randn(kv, 128, generator=g, device="cuda")
        codebook += shift[:, None, None]
        keys += shift[None, :, None]
    if data == "outliers":
        codebook[0, 0, 7], codebook[0, 0, 300, 5], codebook[1, 0, 4000, 100], codebook[1, 0, 9] = 1e12, float("nan"), float("inf"), -1e18
    dims = B.make_dims(1, kv, kv, 128, 1, n_new + 8, n_centroids=4096)
    got = _single(dims, keys, codebook, weights, code, n_new + 8, prepared=True)
    for h in range(kv):
        c, k = codebook[h, 0].double(), keys[0, h].double()
        middle = c[1000:2000].mean(0)
        c, k = c - middle, k - middle
        w = c @ h64[h]
        score = (0.5 * (w * c).sum(-1) - k @ w.t()).nan_to_num(nan=float("inf"), posinf=float("inf"), neginf=float("inf"))
        lost = score.gather(1, got[0, h][:, None])[:, 0] - score.min(1).values
        ordinary = w[1000:2000].norm(dim=1).max()
        assert (lost <= 1e-12 * ((0.5 * (w * c).sum(-1))[1000:2000].max() + k.norm(dim=1) * ordinary)).all(), float(lost.max())
