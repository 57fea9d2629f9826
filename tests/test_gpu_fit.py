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
                                             (1, 1, 50001, True), (12, 1, 60000, False)])   # (of the last: more slices than the scan reads at once)
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


@pytest.mark.parametrize("run", [0, 1, 63, 64, 65, 128, 1000])
@pytest.mark.parametrize("batch,kv,n", [(1, 2, 24577), (7, 3, 14301), (1, 1, 131137), (1, 1, 48000)])
def test_codebook_update_of_runs_across_waves(batch, kv, n, run):
    """Codewords with exactly `run` keys (the last one what is left, 0: all keys one codeword's), so that runs begin and end
    with the waves' shares, span several of them or fill one, and most codewords have no keys."""
    rows = batch * n
    g = torch.Generator(device="cuda").manual_seed(rows + run)
    keys = torch.randn(batch, kv, n, 128, generator=g, device="cuda")
    by_row = torch.zeros(kv, rows, dtype=torch.int64, device="cuda")
    for h in range(kv):
        if run:
            at = torch.arange(rows, device="cuda") // run
            by_row[h] = torch.clamp(at, max=4095 - 2 * h)[torch.randperm(rows, generator=g, device="cuda")]
        else:
            by_row[h] = 4095 - h
    codes = by_row.reshape(kv, batch, n).permute(1, 0, 2).contiguous()
    codebook = torch.randn(kv, 1, 4096, 128, generator=g, device="cuda")
    out = torch.full_like(codebook, float("nan"))
    counts = torch.full((kv, 1, 4096), -1, dtype=torch.int32, device="cuda")
    dims = B.make_dims(batch, kv, kv, 128, 1, n, n_centroids=4096)
    ws = _workspace(dims, False).fill_(0xA5)
    B.codebook_update(dims, keys, n, 0, codes.to(torch.int16).unsqueeze(-1).contiguous(), codebook, out, counts, ws)
    torch.cuda.synchronize()
    for h in range(kv):
        x = keys[:, h].reshape(rows, 128).double()
        sums = torch.zeros(4096, 128, dtype=torch.float64, device="cuda").index_add_(0, by_row[h], x)
        want_n = torch.bincount(by_row[h], minlength=4096)
        assert torch.equal(counts[h, 0].long(), want_n)
        want = torch.where(want_n[:, None] > 0, sums / want_n.clamp(min=1)[:, None], codebook[h, 0].double())
        # one rounding to float32 of sums whose order differs: an ulp where float64 lands next to a midpoint
        assert ((out[h, 0].double() - want).abs() <= 1.2e-7 * want.abs() + 1e-12).all()


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


def _moment(q, kv, least=False):
    heads = q.shape[1]
    dims = B.make_dims(1, heads, kv, 128, 16, 64)
    ws = _workspace(dims, least).fill_(0xFF)
    out = torch.full((kv, 128, 128), float("nan"), device="cuda")
    B.second_moment(dims, q, q.shape[0], out, ws)
    torch.cuda.synchronize()
    for h in range(kv):
        x = q[:, h * (heads // kv):(h + 1) * (heads // kv)].reshape(-1, 128).double()
        yield out[h].double(), x


@pytest.mark.parametrize("heads,kv,n,data", [
    (5, 1, 411, "normal"), (5, 1, 410, "normal"),      # few rows: float64 products
    (5, 1, 3277, "normal"), (5, 1, 3276, "normal"),    # 16385 rows are by digits, 16380 not
    (8, 8, 2049, "normal"), (8, 8, 2047, "normal"),    # 2049 rows of a KV head, 2047
    (7, 1, 1000, "normal"), (7, 1, 3001, "normal"), (6, 2, 5001, "normal"),   # heads that do not divide a step
    (16, 2, 2049, "steps"),                            # values that grow by 2^10 three times: larger units
    (4, 4, 3000, "late"), (4, 4, 9000, "late"),        # dimensions that are zero in the first rows, tiny, or huge
    (8, 1, 2000, "correlated"), (8, 1, 2100, "correlated"),   # equal and opposite dimensions
])
def test_second_moment_by_digits(heads, kv, n, data):
    g = torch.Generator(device="cuda").manual_seed(n)
    q = torch.randn(n, heads, 128, generator=g, device="cuda")
    if data == "steps":
        q *= 1024.0 ** torch.arange(n, device="cuda").mul(4).div(n, rounding_mode="floor")[:, None, None]
    if data == "late":
        q[:n // 2, :, :20] = 0
        q[..., 20:40] *= 1e-17
        q[..., 40:50] *= 1e15
        q[..., 50] = 0
    if data == "correlated":
        q[..., 1], q[..., 2] = q[..., 0], -q[..., 0]
    for got, x in _moment(q, kv):
        want = x.t() @ x / x.shape[0]
        # half an ulp of float32, and of the sum of magnitudes what the digits may leave out (see the next test)
        assert ((got - want).abs() <= 6e-8 * want.abs() + 2e-10 * (x.abs().t() @ x.abs()) / x.shape[0] + 1e-45).all()
        assert torch.equal(got, got.t())


@pytest.mark.parametrize("factor", [30.0, 1e3, 1e4, 1e6, 1e12])
@pytest.mark.parametrize("heads,kv,n,data", [
    (4, 1, 4097, "one row each"), (8, 2, 3073, "one row each"), (4, 1, 20000, "last"), (4, 4, 60000, "first"),
    (5, 1, 30011, "tenth"), (8, 1, 9000, "heads"), (4, 1, 9000, "heavy")])
def test_second_moment_of_a_few_large_values(factor, heads, kv, n, data):
    """Rows that are large in one dimension where another is not: H_ij comes from the many small products, which float64
    sums keep."""
    g = torch.Generator(device="cuda").manual_seed(n)
    q = torch.randn(n, heads, 128, generator=g, device="cuda")
    q[..., 90] += 0.5 * q[..., 3]
    if data == "one row each":
        q[n // 3, 0, 3] *= factor
        q[n // 2, -1, 90] *= factor
        q[n - 1, :, 17] *= factor
    if data == "last":                               # at the end of the workgroups' shares
        q[n // 8 - 1::n // 8, :, 3] *= factor
        q[n // 8 - 2::n // 8, :, 90] *= factor
    if data == "first":
        q[::n // 32, :, 3:60] *= factor
        q[1::n // 32, :, 60:] *= factor
    if data == "tenth":                              # large in one dimension or in the other, not in both
        rows = torch.rand(n, 1, generator=g, device="cuda")
        q[..., 3] *= torch.where(rows < 0.1, factor, 1.0)
        q[..., 90] *= torch.where(rows > 0.9, factor, 1.0)
    if data == "heads":
        q[:, 1::2, ::2] *= factor
        q[:, ::2, 1::2] *= factor
    if data == "heavy":                              # no variance at all
        q /= torch.randn(n, heads, 128, generator=g, device="cuda").abs() + 1.0 / factor
    for got, x in _moment(q, kv):
        want = x.t() @ x / x.shape[0]
        # Half an ulp of float32, and what the digits leave out: 0.2 a row, of either sign, where the rows' |V_i V_j| are 2^27
        # or more on average: 1.5e-9 / sqrt(rows) of their sum, five times that from 2048 rows on.
        assert ((got - want).abs() <= 6e-8 * want.abs() + 2e-10 * (x.abs().t() @ x.abs()) / x.shape[0]).all()
        assert torch.equal(got, got.t())


@pytest.mark.parametrize("n", [3000, 9000])   # float64 products, digits
def test_second_moment_of_values_that_are_not_finite(n):
    q = torch.randn(n, 4, 128, generator=torch.Generator(device="cuda").manual_seed(1), device="cuda")
    q[n - 1, 0, 3] = float("nan")     # head 0: the last row
    q[0, 1, 5] = float("inf")         # head 1: the first
    q[n // 2, 1, 9] = float("-inf")
    q[n // 2, 2, 77] = float("inf")   # head 2: in the middle; head 3: none
    for got, x in _moment(q, 4):
        want = x.t() @ x / x.shape[0]
        assert torch.equal(got.isnan(), want.isnan()) and torch.equal(got.isinf(), want.isinf())
        ok = want.isfinite()
        assert torch.equal(got[want.isinf()], want[want.isinf()])
        assert ((got - want).abs()[ok] <= 6e-8 * want.abs()[ok] + 1e-11).all()


def test_second_moment_of_long_shares():
    """More rows to a workgroup than its 32-bit sums hold, in the least workspace."""
    q = torch.randn(1900000, 1, 128, generator=torch.Generator(device="cuda").manual_seed(2), device="cuda")
    q[..., 7] = 3.0                                    # the digits' products all of one sign
    for got, x in _moment(q, 1, least=True):
        want = x.t() @ x / x.shape[0]
        assert ((got - want).abs() <= 6e-8 * want.abs() + 1e-13).all()
