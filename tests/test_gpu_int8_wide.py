"""The int8 GEMM on tiles of 128 tokens x 256 and 192 columns, 256 x 128 and 128 x 128 of eight waves: every tile and K split that
a weight form has, at the edges of tokens, columns and chunks and with a second round of workgroups, against the product in
float64 of the stored codes."""
import pytest
import torch

from paper_2506_10443_amd import binding as B

pytestmark = pytest.mark.gpu

FORMS = {"w4": B.MODE_W4_ZP_INT, "w4min": B.MODE_W4_MIN_FLOAT, "w8": B.MODE_W8_MIN_FLOAT | B.NATIVE_8BIT}
TILES = {"w4": ("x1", "x1k", "c1", "c1k", "w1", "v1"), "w4min": ("s1", "s1k", "v1k"), "w8": ("x1", "x1k", "c1", "c1k", "s1", "v1")}
# one chunk, and an odd number of chunks (the minima go two chunks at a time); one row tile; one past a tile and one short of it;
# K split into unequal parts; many tiles of an odd number of rows; and more than two workgroups per CU of 256 CUs - 531 tiles of
# 128 x 256, 295 of 256 x 128, two on a CU at a time - ragged in both directions
SHAPES = [(128, 256, 128), (17, 16, 384), (129, 272, 640), (255, 208, 1152), (300, 784, 1152), (1030, 1040, 384), (1030, 14864, 384)]
HALF_CHUNK = [(130, 272, 192), (77, 16, 320), (128, 256, 64)]      # an odd number of groups (4-bit codes only)


@pytest.mark.parametrize("form,M,N,K", [(f, *s) for f in FORMS for s in SHAPES + (HALF_CHUNK if f != "w8" else [])])
def test_wide_tiles_match_exact(form, M, N, K):
    print("int8 wide", form, M, N, K, flush=True)
    mode = FORMS[form]
    gen = torch.Generator(device="cuda:0").manual_seed(M + N + K)
    W = torch.randn((N, K), generator=gen, device="cuda:0") * 0.02
    W[0, :64] = 0.25                      # a constant group: step 1, far from what its neighbours hold
    W[N - 1] = 0.0
    packed = B.mnnq_pack_weights(W, mode=mode)
    x = torch.randn((M, K), generator=gen, device="cuda:0")
    x[:, 5] *= 20.0
    x[M // 2] = 0.0
    bias = torch.randn(N, generator=gen, device="cuda:0")
    xq, sx, _ = B.mnnq_quant_act(x, want_xsum=False)
    q, s, z = (t.double() for t in B.mnnq_unpack_weights(packed, N, K, mode=mode))
    q, s, z = q.view(N, K // 64, 64), s[:, :, None], z[:, :, None]
    w = ((q - z) * s if form == "w4" else q * s + z).view(N, K)
    exact = (xq.double() @ w.t()) * sx.double()[:, None] + bias.double()
    for tile in TILES[form] + (None,):      # (None: the kernel that the shape takes)
        out = torch.full((M + 1, N), float("nan"), device="cuda:0")
        B.mnnq_debug_set("MNNQ_PREFILL_TILE", tile)
        B.mnnq_debug_set("MNNQ_NO_SKINNY", None if tile is None else 1)
        try:
            y = B.mnnq_linear_prefill(packed, N, K, xq, sx, bias=bias, out=out[:M], mode=mode)
            half = B.mnnq_linear_prefill_o16(packed, N, K, xq, sx, bias=bias, mode=mode)
        finally:
            B.mnnq_debug_set("MNNQ_PREFILL_TILE", None)
            B.mnnq_debug_set("MNNQ_NO_SKINNY", None)
        assert torch.isnan(out[M]).all(), tile
        assert (y.double() - exact).abs().max() <= 1e-5 * exact.abs().max(), tile      # the layer's tolerance
        assert torch.equal(half, y.half()), tile


def test_the_tile_follows_the_shape():
    plan = lambda m, n, k, f: B.mnnq_plan_debug(4, m, n, k, FORMS[f])[:4]
    assert plan(1024, 37888, 3584, "w8") == [0, 128, 256, 4] and plan(333, 28672, 4096, "w8") == [0, 128, 192, 4]
    assert plan(1024, 37888, 3584, "w4min") == [0, 128, 128, 4] and plan(384, 37888, 3584, "w4") == [0, 128, 256, 4]
