"""The calibration kernels against float64 sums, at the sizes where their splits could go wrong."""
import pytest
import torch

from paper_2502_12665_amd import binding as B

pytestmark = pytest.mark.gpu


def _workspace(dims, least):
    """What the fastest forms ask for, or no more than the 8 MiB per KV head that any size of call can do with."""
    n = B.workspace_bytes(dims, B.OP_FIT)
    return torch.empty(min(n, dims.n_kv_heads << 23) if least else n, dtype=torch.uint8, device="cuda")


@pytest.mark.parametrize("m", [1, 16, 32])
@pytest.mark.parametrize("least", [False, True])
@pytest.mark.parametrize("batch,kv,n,skew", [(1, 1, 1, False), (2, 3, 63, False), (1, 2, 4097, True), (3, 8, 2050, False),
                                             (1, 1, 50001, True), (12, 1, 60000, False)])
def test_codebook_update(m, least, batch, kv, n, skew):
    L, ds, stride, pos0 = (4096, 128, n + 9, 5) if m == 1 else (256, 128 // m, n + 9, 5)
    g = torch.Generator(device="cuda").manual_seed(n + m)
    keys = torch.randn(batch, kv, n, 128, generator=g, device="cuda")
    codes = torch.randint(0, L, (batch, kv, stride, m), generator=g, device="cuda")
    if skew:                                                  # nine tenths of the keys share three codes
        few = torch.rand(codes.shape, generator=g, device="cuda") < 0.9
        codes = torch.where(few, codes % 3, codes)
    codebook = torch.randn(kv, m, L, ds, generator=g, device="cuda")
    out = torch.full_like(codebook, float("nan"))
    counts = torch.full((kv, m, L), -1, dtype=torch.int32, device="cuda")
    dims = B.make_dims(batch, kv, kv, 128, m, stride, n_centroids=L)
    ws = _workspace(dims, least).fill_(0xA5)
    B.codebook_update(dims, keys, n, pos0, codes.to(torch.int16 if m == 1 else torch.uint8), codebook, out, counts, ws)
    torch.cuda.synchronize()
    used = codes[:, :, pos0:pos0 + n]
    sums = torch.zeros(kv, m, L, ds, dtype=torch.float64, device="cuda")
    want_n = torch.zeros(kv, m, L, dtype=torch.int64, device="cuda")
    for h in range(kv):
        for s in range(m):
            c = used[:, h, :, s].reshape(-1)
            sums[h, s].index_add_(0, c, keys[:, h, :, s * ds:(s + 1) * ds].reshape(-1, ds).double())
            want_n[h, s] = torch.bincount(c, minlength=L)
    assert torch.equal(counts.long(), want_n)
    mean = sums / want_n.clamp(min=1)[..., None]
    want = torch.where(want_n[..., None] > 0, mean, codebook.double())
    # one rounding to float32 of sums whose order differs: an ulp where float64 lands next to a midpoint
    assert ((out.double() - want).abs() <= 1.2e-7 * want.abs() + 1e-12).all()


@pytest.mark.parametrize("heads,kv,n", [(8, 1, 1), (5, 1, 13), (6, 2, 1025), (7, 1, 4800), (24, 3, 3001), (64, 64, 40), (8, 1, 4096)])
@pytest.mark.parametrize("least", [False, True])
def test_second_moment_shares(heads, kv, n, least):
    g = torch.Generator(device="cuda").manual_seed(n)
    q = torch.randn(n, heads, 128, generator=g, device="cuda") * torch.linspace(0.1, 4.0, 128, device="cuda")
    dims = B.make_dims(1, heads, kv, 128, 16, 64)
    ws = _workspace(dims, least).fill_(0xFF)   # (NaN)
    out = torch.full((kv, 128, 128), float("nan"), device="cuda")
    B.second_moment(dims, q, n, out, ws)
    torch.cuda.synchronize()
    for h in range(kv):
        x = q[:, h * (heads // kv):(h + 1) * (heads // kv)].reshape(-1, 128).double()
        want = x.t() @ x / x.shape[0]
        scale = torch.sqrt(torch.diagonal(want)[:, None] * torch.diagonal(want)[None])
        assert ((out[h].double() - want).abs() <= 6e-8 * want.abs() + 1e-13 * scale).all()
        assert torch.equal(out[h], out[h].t())
