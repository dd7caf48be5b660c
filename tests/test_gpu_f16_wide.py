"""The fp16-activation GEMM on tiles of 128 tokens x 256, 192 and 128 columns: every tile and K split, at the edges of tokens,
columns and groups."""
import pytest
import torch

from paper_2506_10443_amd import binding as B

pytestmark = pytest.mark.gpu

# one group; an odd number of groups (a padding group, whose activations would be the next token's); fewer chunks than K parts;
# one row tile; columns and tokens one past a tile, one short of it; an odd number of rows of tiles; more than two workgroups per
# CU of 256 CUs, ragged in both directions
SHAPES = [(128, 256, 64), (129, 16, 192), (127, 272, 320), (257, 208, 448), (300, 784, 1088), (17, 528, 2176), (1030, 1040, 384),
          (1030, 14864, 384)]


@pytest.mark.parametrize("M,N,K", SHAPES)
@pytest.mark.parametrize("tile", ["b1", "b1k", "c1", "c1k", "d1", None])      # (None: the kernel that the shape takes)
def test_wide_tiles_match_exact(tile, M, N, K):
    print("fp16 wide", tile, M, N, K, flush=True)
    gen = torch.Generator(device="cuda:0").manual_seed(M + N + K)
    packed = B.mnnq_pack_weights(torch.randn((N, K), generator=gen, device="cuda:0") * 0.02)
    x = torch.randn((M, K), generator=gen, device="cuda:0").half()
    q, s, z = (t.double() for t in B.mnnq_unpack_weights(packed, N, K))
    w = ((q.view(N, K // 64, 64) - z[:, :, None]) * s[:, :, None]).view(N, K)
    bias, rs = (torch.randn(n, generator=gen, device="cuda:0") for n in (N, M))
    product = x.double() @ w.t()
    out = torch.full((M + 1, N), float("nan"), device="cuda:0")
    x_inf = x.clone()
    x_inf[M // 2] = float("inf")          # infinities stay in their own token's row
    B.mnnq_debug_set("MNNQ_PREFILL_TILE", tile)
    B.mnnq_debug_set("MNNQ_NO_SKINNY", None if tile is None else 1)
    try:
        y = B.mnnq_linear_prefill_f16(packed, N, K, x, bias=bias, out=out[:M])
        half = B.mnnq_linear_prefill_f16_o16(packed, N, K, x, bias=bias)
        scaled = B.mnnq_linear_prefill_f16(packed, N, K, x, row_scale=rs)
        y_inf = B.mnnq_linear_prefill_f16(packed, N, K, x_inf, bias=bias)
    finally:
        B.mnnq_debug_set("MNNQ_PREFILL_TILE", None)
        B.mnnq_debug_set("MNNQ_NO_SKINNY", None)
    assert torch.isnan(out[M]).all()      # nothing behind the last token
    exact = product + bias.double()
    assert (y.double() - exact).abs().max() <= 1e-5 * exact.abs().max()     # fp32 sums: the layer's tolerance
    assert torch.equal(half, y.half())
    exact = product * rs.double()[:, None]
    assert (scaled.double() - exact).abs().max() <= 1e-5 * exact.abs().max()
    rows = torch.arange(M, device="cuda:0") != M // 2
    assert torch.equal(y_inf[rows], y[rows]) and not torch.isfinite(y_inf[M // 2]).any()


def test_the_tile_follows_the_shape():
    """Each tile is what some shape takes without a switch (256 CUs), the K-split kernel where tiles are few."""
    plan = lambda m, n, k: B.mnnq_plan_debug(5, m, n, k, B.MODE_W4_ZP_INT)[:5]
    assert plan(2048, 28672, 4096) == [0, 128, 256, 4, 4]
    assert plan(2048, 4096, 14336) == [0, 128, 256, 8, 8]
    assert plan(2048, 6144, 4096) == [0, 128, 192, 4, 4]
    assert plan(1024, 6144, 4096) == [0, 128, 192, 8, 8]
    assert plan(1024, 4096, 14336) == [0, 128, 128, 8, 8]
    assert plan(512, 1536, 8960)[0] == 3
