"""Imported scales and minima that are infinite, NaN, or so large that `minimum + middle code * scale` overflows: the kernels that
centre the codes give the sum over the groups of scale * (sum x q) + minimum * (sum x), infinity for infinity, and the other weight rows
are untouched."""
import pytest
import torch

from paper_2506_10443_amd import binding as B

pytestmark = pytest.mark.gpu

W8N = B.MODE_W8_MIN_FLOAT | B.NATIVE_8BIT
INF, NAN = float("inf"), float("nan")
# row -> (group, scale, minimum): None leaves what the group holds.  A code sum of 1 keeps 2e37 (3e37 with fp16) finite, the middle does not.
EXTREMES = {3: (0, INF, None), 17: (1, -INF, None), 20: (2, NAN, None), 35: (3, None, INF), 36: (0, None, -INF), 40: (1, 2e37, None),
            41: (3, 3.4e37, None), 55: (2, INF, -INF)}


def _case(mode, N, K, seed):
    gen = torch.Generator(device="cuda:0").manual_seed(seed)
    top = 256 if mode == W8N else 16
    q = torch.randint(0, top, (N, K), generator=gen, device="cuda:0", dtype=torch.uint8)
    s = torch.rand((N, K // 64), generator=gen, device="cuda:0") * 0.01 + 1e-3
    mn = -s * (top / 2)
    for n, (g, scale, low) in EXTREMES.items():
        if scale is not None:
            s[n, g] = scale
        if low is not None:
            mn[n, g] = low
    q[40:42] = 1        # (rows 40 and 41: the products of a one-hot token stay finite)
    return B.mnnq_pack_from_quantized(q, s, mn, mode=mode), q, s, mn, gen


def _definition(x, q, s, mn):
    """Group by group in binary32, the products' sums exact (integers) or rounded once."""
    y = torch.zeros((x.shape[0], q.shape[0]), device="cuda:0")
    for g in range(s.shape[1]):
        xg = x[:, 64 * g:64 * g + 64].double()
        y += s[:, g] * (xg @ q[:, 64 * g:64 * g + 64].double().t()).float()
        y += mn[:, g] * xg.sum(1, keepdim=True).float()
    return y


def _same(y, want, rows):
    assert torch.equal(torch.isnan(y), torch.isnan(want))
    assert torch.equal(torch.isposinf(y), torch.isposinf(want)) and torch.equal(torch.isneginf(y), torch.isneginf(want))
    ok = torch.isfinite(want)
    # fp32 sums, bounded by each row's largest value as everywhere (the extreme rows have a scale of their own)
    for part in (rows, ~rows):
        f = torch.where(ok, want, 0.0)[:, part]
        assert ((torch.where(ok, y, 0.0)[:, part] - f).abs() <= 1e-5 * f.abs().amax()).all()


# K-split kernel (rows; fused: token blocks) of all four tile heights and both numbers of waves, wide tiles whole and split
@pytest.mark.parametrize("M,tile", [(20, None), (40, None), (70, None), (150, None), (300, None), (300, "x1"), (300, "x1k"), (300, "c1"), (300, "c1k")])
def test_int8_bytes(M, tile):
    print("extremes, bytes", M, tile, flush=True)
    N, K = 528, 1024
    packed, q, s, mn, gen = _case(W8N, N, K, 7 + M)
    x = torch.randn((M, K), generator=gen, device="cuda:0")
    x[1] = 0.0
    x[2] = 0.0
    x[2, 70] = 1.0      # one-hot tokens, in groups 1 and 3
    x[3] = 0.0
    x[3, 200] = -1.0
    xq, sx, _ = B.mnnq_quant_act(x, want_xsum=False)
    xq[2:4] = torch.sign(xq[2:4])
    want = _definition(xq, q, s, mn) * sx[:, None]
    rows = torch.zeros(N, dtype=torch.bool, device="cuda:0")
    rows[list(EXTREMES)] = True
    B.mnnq_debug_set("MNNQ_PREFILL_TILE", tile)
    try:
        _same(B.mnnq_linear_prefill(packed, N, K, xq, sx, mode=W8N), want, rows)
    finally:
        B.mnnq_debug_set("MNNQ_PREFILL_TILE", None)
    if tile is None:
        xr = x.clone()
        xr[2:4] = 0.0   # (a one-hot token's only code is 127)
        xq, sx, _ = B.mnnq_quant_act(xr, want_xsum=False)
        want = _definition(xq, q, s, mn) * sx[:, None]
        _same(B.mnnq_linear_prefill_fused(packed, N, K, xr, mode=W8N), want, rows)


@pytest.mark.parametrize("M", [20, 40, 70, 150, 300])
def test_fp16_activations(M):
    print("extremes, fp16", M, flush=True)
    N, K, mode = 528, 960, B.MODE_W4_MIN_FLOAT     # an odd number of groups
    packed, q, s, mn, gen = _case(mode, N, K, 9 + M)
    x = torch.randn((M, K), generator=gen, device="cuda:0").half()
    x[1:4] = 0.0
    x[2, 70] = 1.0
    x[3, 200] = -1.0
    want = _definition(x, q, s, mn)
    rows = torch.zeros(N, dtype=torch.bool, device="cuda:0")
    rows[list(EXTREMES)] = True
    _same(B.mnnq_linear_prefill_f16(packed, N, K, x, mode=mode), want, rows)
