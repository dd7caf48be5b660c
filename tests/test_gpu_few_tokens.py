"""Few tokens at once (the kernels behind mnnq_linear_prefill and mnnq_linear_prefill_fused for small M) against the
oracle: token counts at the edges of the 16-token blocks, rows of one chunk, of an odd number of groups and beyond what a
wave holds in registers, one and several row tiles per workgroup, every weight form.  int8 rows given (row-major)
and quantized by the call (codes in token blocks) run the same sums in the same order: equal bit for bit."""
import numpy as np
import pytest
import torch

import oracle
from paper_2506_10443_amd import binding as B, synth

pytestmark = pytest.mark.gpu
W8N = B.MODE_W8_MIN_FLOAT | B.NATIVE_8BIT
FORMS = {
    "w4": (B.MODE_W4_ZP_INT, oracle.quant_weights, oracle.linear_w4a8),
    "w4min": (B.MODE_W4_MIN_FLOAT, oracle.quant_weights_minf, oracle.linear_w4a8_minf),
    "w8": (W8N, oracle.quant_weights8, oracle.linear_w8a8),
    "w8planes": (B.MODE_W8_MIN_FLOAT, oracle.quant_weights8, oracle.linear_w8a8),
}
# (M, N, K): the last ones have many row tiles, one per workgroup, and stream a long row
SHAPES = [(2, 16, 64), (3, 48, 192), (15, 80, 1536), (16, 32, 4096), (17, 48, 4160), (32, 64, 960), (33, 48, 512),
          (48, 32, 8960), (49, 16, 320), (64, 80, 3584), (4, 16 * 1100, 128), (40, 16 * 600, 256), (5, 32, 18944),
          (2, 16, 24576), (81, 48, 1536), (128, 32, 320)]


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


@pytest.mark.parametrize("M,N,K", SHAPES)
@pytest.mark.parametrize("form", list(FORMS))
def test_few_tokens_match_oracle(form, M, N, K):
    mode, quant, linear = FORMS[form]
    if form.startswith("w8") and K % 128:
        pytest.skip("int8 weights: K a multiple of 128")
    print("few tokens", form, M, N, K, flush=True)
    W = synth.weights(N, K, 3000 + M + N + K)
    W[0, :64] = 0.25                                # a constant group
    x = synth.activations(M, K, 3001 + M + N + K)
    x[M // 2] = 0.0                                 # a zero token
    q, s, z = quant(W)
    xq, sx, _ = oracle.quant_act(x)
    bias = synth.weights(1, N, 9)[0] * 10
    y_o = linear(xq, sx, q, s, z, bias=bias, want_acc=False)[1]
    packed = B.mnnq_pack_weights(dev(W), mode=mode)
    bd, xd = dev(bias), dev(x)
    y = B.mnnq_linear_prefill(packed, N, K, dev(xq), dev(sx), bias=bd, mode=mode)
    # fp32 sums of up to 2 K / 64 group terms: the layer's tolerance
    assert np.abs(y.cpu().numpy() - y_o).max() <= 1e-5 * np.abs(y_o).max()
    out = torch.full((M + 1, N), float("nan"), device="cuda:0")
    yf = B.mnnq_linear_prefill_fused(packed, N, K, xd, bias=bd, out=out[:M], mode=mode)
    assert torch.isnan(out[M]).all()                # nothing behind the last token
    assert torch.equal(yf, y)
    assert np.abs(yf.cpu().numpy() - y_o).max() <= 1e-5 * np.abs(y_o).max()
    y16 = B.mnnq_linear_prefill_fused_o16(packed, N, K, xd, bias=bd, mode=mode)
    assert torch.equal(y16, yf.half())


@pytest.mark.parametrize("M", [2, 17, 33, 49])
@pytest.mark.parametrize("N,K", [(48, 640), (16 * 600, 320), (64, 1152), (32, 3136)])
def test_few_tokens_extreme_codes_and_uneven_waves(M, N, K):
    """Waves with fewer chunks than they have room for (5, 3, 9 and 25 chunks, odd rows among them), tokens whose codes are all -128
    or all 127, zero points 0 and 15: the starts of the accumulators are as large as they get."""
    print("few tokens, extreme codes", M, N, K, flush=True)
    rng = np.random.default_rng(M + N + K)
    W = synth.weights(N, K, 41)
    W[0] = np.abs(W[0]) + 0.01                      # minimum above zero: zero point 0
    W[1] = -np.abs(W[1]) - 0.01                     # maximum below zero: zero point 15
    q, s, z = oracle.quant_weights(W)
    xq = rng.integers(-128, 128, (M, K)).astype(np.int8)
    xq[0], xq[M - 1] = -128, 127
    sx = rng.uniform(0.001, 0.1, M).astype(np.float32)
    y_o = oracle.linear_w4a8(xq, sx, q, s, z, want_acc=False)[1]
    packed = B.mnnq_pack_weights(dev(W), mode=B.MODE_W4_ZP_INT)
    y = B.mnnq_linear_prefill(packed, N, K, dev(xq), dev(sx), mode=B.MODE_W4_ZP_INT).cpu().numpy()
    # fp32 sums of up to K / 64 group terms: the layer's tolerance, token by token
    assert (np.abs(y - y_o).max(axis=1) <= 1e-5 * np.abs(y_o).max(axis=1)).all()


@pytest.mark.parametrize("M,N,K", [(33, 32, 64), (65, 48, 192), (100, 64, 4160), (130, 272, 3584), (257, 32, 18944)])
def test_quantizer_writes_the_planes_of_the_two_steps(M, N, K):
    """The fused call on a buffer with the matrix-core plane: bit for bit the result of quantizer, planes and GEMM as
    calls of their own (the quantizer writes the operand planes itself)."""
    mode = B.MODE_W4_ZP_INT | B.WITH_MATRIX_PLANE
    print("fused planes", M, N, K, flush=True)
    packed = B.mnnq_pack_weights(dev(synth.weights(N, K, 3100 + K)), mode=mode)
    xd = dev(synth.activations(M, K, 3101 + M))
    B.mnnq_debug_set("MNNQ_PREFILL6_PLAN", 0)       # (shapes this small are left to other kernels)
    try:
        yf = B.mnnq_linear_prefill_fused(packed, N, K, xd, mode=mode)
        xq, sx, _ = B.mnnq_quant_act(xd)
        y = B.mnnq_linear_prefill_planes(packed, M, N, K, B.mnnq_act_planes(xq), sx, mode=mode)
    finally:
        B.mnnq_debug_set("MNNQ_PREFILL6_PLAN", None)
    assert torch.equal(yf, y)


# K split over the waves (65 tokens and more on layers too large for the few-token kernels): fewer chunks than waves, odd
# shares, rows and columns past the tile, an odd number of groups, one and several tiles per CU
GEMM_SHAPES = [(129, 48, 64), (130, 16, 192), (192, 80, 1088), (333, 272, 1536), (200, 1040, 640), (65, 16 * 520, 2048),
               (700, 16 * 60, 256), (129, 32, 8960)]


@pytest.mark.parametrize("M,N,K", GEMM_SHAPES)
@pytest.mark.parametrize("form", ["w4", "w4min", "w8"])
def test_k_split_int8_gemm_matches_oracle(form, M, N, K):
    mode, quant, linear = FORMS[form]
    if form == "w8" and K % 128:
        pytest.skip("int8 weights: K a multiple of 128")
    print("K-split int8 GEMM", form, M, N, K, flush=True)
    W = synth.weights(N, K, 3200 + M + N + K)
    W[0, :64] = 0.25                                # a constant group
    x = synth.activations(M, K, 3201 + M + N + K)
    x[M // 2] = 0.0                                 # a zero token
    q, s, z = quant(W)
    xq, sx, _ = oracle.quant_act(x)
    bias = synth.weights(1, N, 9)[0] * 10
    y_o = linear(xq, sx, q, s, z, bias=bias, want_acc=False)[1]
    tol = 1e-5 * np.abs(y_o).max()
    packed = B.mnnq_pack_weights(dev(W), mode=mode)
    bd, xd = dev(bias), dev(x)
    out = torch.full((M + 1, N), float("nan"), device="cuda:0")
    y = B.mnnq_linear_prefill(packed, N, K, dev(xq), dev(sx), bias=bd, out=out[:M], mode=mode)
    assert torch.isnan(out[M]).all()                # nothing behind the last token
    assert np.abs(y.cpu().numpy() - y_o).max() <= tol
    yf = B.mnnq_linear_prefill_fused(packed, N, K, xd, bias=bd, mode=mode)
    assert torch.equal(yf, y)
    assert torch.equal(B.mnnq_linear_prefill_fused_o16(packed, N, K, xd, bias=bd, mode=mode), yf.half())


# fp16 activations: the few-token kernels (resident and streaming, both slices) and the K-split GEMM behind them
F16_SHAPES = [(2, 16, 64), (15, 80, 1536), (16, 32, 8960), (17, 48, 4160), (33, 48, 1984), (40, 16 * 300, 2304), (64, 80, 2048),
              (100, 48, 1536), (65, 48, 192), (130, 272, 1088), (3, 16 * 1100, 128), (6, 16 * 515, 2176), (200, 1040, 640), (129, 32, 8960), (65, 16 * 520, 2048)]


@pytest.mark.parametrize("M,N,K", F16_SHAPES)
@pytest.mark.parametrize("form", ["w4", "w4min", "w8planes"])
def test_fp16_activations_match_oracle(form, M, N, K):
    mode, quant, _ = FORMS[form]
    if form == "w8planes" and K % 128:
        pytest.skip("int8 weights: K a multiple of 128")
    print("fp16 activations", form, M, N, K, flush=True)
    W = synth.weights(N, K, 3300 + M + N + K)
    W[0, :64] = 0.25                                # a constant group
    x16 = synth.activations_f16(M, K, 3301 + M + N + K, outliers=True)
    q, s, z = quant(W)
    bias = synth.weights(1, N, 9)[0] * 10
    linear = oracle.linear_w4a16 if form == "w4" else oracle.linear_a16_minf
    y_o = linear(x16, q, s, z, bias=bias)
    # exact products, fp32 sums of 64 products and then of up to 2 K / 64 groups
    tol = 1e-5 * np.abs(y_o).max()
    packed = B.mnnq_pack_weights(dev(W), mode=mode)
    bd, xd = dev(bias), dev(x16)
    out = torch.full((M + 1, N), float("nan"), device="cuda:0")
    y = B.mnnq_linear_prefill_f16(packed, N, K, xd, bias=bd, out=out[:M], mode=mode)
    assert torch.isnan(out[M]).all()                # nothing behind the last token
    assert np.abs(y.cpu().numpy() - y_o).max() <= tol
    assert torch.equal(B.mnnq_linear_prefill_f16_o16(packed, N, K, xd, bias=bd, mode=mode), y.half())
    rs = np.linspace(0.5, 2.0, M).astype(np.float32)
    y_rs = linear(x16, q, s, z) * rs[:, None].astype(np.float64)
    yr = B.mnnq_linear_prefill_f16(packed, N, K, xd, row_scale=dev(rs), mode=mode).cpu().numpy()
    assert np.abs(yr - y_rs).max() <= 2 * tol


@pytest.mark.parametrize("K", [64, 2112, 20480])
@pytest.mark.parametrize("M", [5, 8, 9, 64, 65, 256, 257, 330])
def test_quantizer_row_sets(M, K):
    """The packing quantizer deals sets of 64 rows to workgroups, one or two rows each (the line at 256): every row is
    quantized and nothing past the last one, at the edges of sets and of the shortest and longest rows it holds."""
    print("quantizer rows", M, K, flush=True)
    x = dev(synth.activations(M, K, 77 + M))
    xq, sx, _ = B.mnnq_quant_act(x)
    forms = [B.MODE_W4_ZP_INT] + ([W8N] if K % 128 == 0 else [])
    for mode in forms:
        packed = B.mnnq_pack_weights(dev(synth.weights(32, K, 78)), mode=mode)
        rows = B.mnnq_linear_prefill(packed, 32, K, xq, sx, mode=mode)
        out = torch.full((M + 1, 32), float("nan"), device="cuda:0")
        B.mnnq_linear_prefill_fused(packed, 32, K, x, out=out[:M], mode=mode)
        assert torch.equal(out[:M], rows) and torch.isnan(out[M]).all()


@pytest.mark.parametrize("K", [64, 3584, 20480, 20544])
def test_two_kernel_decode(K):
    """The fused one-token call with its quantizer as a kernel of its own (large layers; here forced): the packing
    quantizer up to 20480 values, the row-splitting one beyond, both as the separate calls."""
    print("two-kernel decode", K, flush=True)
    x = dev(synth.activations(1, K, 79))
    packed = B.mnnq_pack_weights(dev(synth.weights(48, K, 80)))
    xq, sx, _ = B.mnnq_quant_act(x)
    ws = torch.empty(B.mnnq_workspace_size(1, 48, K), dtype=torch.uint8, device="cuda:0")
    B.mnnq_debug_set("MNNQ_FUSED_TWO_KERNEL_MIB", 0)
    try:
        y = B.mnnq_linear_decode_fused(packed, 48, K, x[0].contiguous(), workspace=ws)
    finally:
        B.mnnq_debug_set("MNNQ_FUSED_TWO_KERNEL_MIB", None)
    assert torch.equal(y, B.mnnq_linear_decode(packed, 48, K, xq[0].contiguous(), sx))


# one shape per tile height of the K-split kernel (16, 32, 48, 64 rows) and number of waves, ragged in rows and columns, the
# tall ones in one round and in two; and two shapes whose rounds are too short for it
HEIGHTS = [(131, 1040, 320, 16, 8), (131, 2064, 320, 32, 8), (200, 4112, 320, 32, 4), (500, 1040, 320, 48, 8), (333, 4080, 192, 48, 4),
           (200, 4080, 320, 64, 8), (500, 4080, 320, 64, 4), (500, 4112, 192, 0, 0), (1100, 4096, 128, 0, 0)]


@pytest.mark.parametrize("M,N,K,height,waves", HEIGHTS)
@pytest.mark.parametrize("form", ["w4", "w4min", "w8"])
def test_k_split_tile_heights(form, M, N, K, height, waves):
    mode, quant, linear = FORMS[form]
    if form == "w8":
        K = (K + 127) // 128 * 128
    for what in (4,) if form == "w8" else (4, 5):       # the kernel that runs (5: with fp16 activations)
        plan = B.mnnq_plan_debug(what, M, N, K, mode)
        assert plan[:4] == [3, height, 64, waves] if height else plan[0] == 0
    print("K-split heights", form, M, N, K, flush=True)
    W, x = synth.weights(N, K, 3300 + M), synth.activations(M, K, 3301 + M)
    q, s, z = quant(W)
    xq, sx, _ = oracle.quant_act(x)
    bias = synth.weights(1, N, 9)[0] * 10
    y_o = linear(xq, sx, q, s, z, bias=bias, want_acc=False)[1]
    packed = B.mnnq_pack_weights(dev(W), mode=mode)
    out = torch.full((M + 1, N), float("nan"), device="cuda:0")
    B.mnnq_linear_prefill_fused(packed, N, K, dev(x), bias=dev(bias), out=out[:M], mode=mode)
    assert torch.isnan(out[M]).all()
    assert np.abs(out[:M].cpu().numpy() - y_o).max() <= 1e-5 * np.abs(y_o).max()
    # int8 rows, whose pieces the kernel exchanges between its lanes: the same sums in the same order
    assert torch.equal(B.mnnq_linear_prefill(packed, N, K, dev(xq), dev(sx), bias=dev(bias), mode=mode), out[:M])
    if form != "w8":        # fp16 activations: fp32 sums as the tiled kernel's, in another order
        x16 = dev(synth.activations_f16(M, K, 3302 + M))
        y16 = B.mnnq_linear_prefill_f16(packed, N, K, x16, mode=mode)
        B.mnnq_debug_set("MNNQ_NO_SKINNY", 1)
        try:
            ref = B.mnnq_linear_prefill_f16(packed, N, K, x16, mode=mode)
        finally:
            B.mnnq_debug_set("MNNQ_NO_SKINNY", None)
        assert (y16 - ref).abs().max() <= 1e-5 * ref.abs().max()


# The fp16 GEMM's tile by tiles per CU (three rows of 128-row tiles, two of 256-row tiles, 86 columns on 256 CUs): one
# 256 x 128 tile split over K where the rows are long (an odd number of groups, so that the halves differ, among them), two
# of 128 x 128 where they are short or one column too many makes a second tile.  (1100 and 20000 columns: one and four)
@pytest.mark.parametrize("M,N,K", [(380, 10992, 3072), (380, 10992, 3136), (380, 10992, 3008), (380, 16400, 3072),
                                   (257, 1104, 3136), (513, 26608, 192)])
@pytest.mark.parametrize("mode", [B.MODE_W4_ZP_INT, B.MODE_W4_MIN_FLOAT])
def test_fp16_tiles_by_tiles_per_cu(mode, M, N, K):
    print("fp16 tiles", mode, M, N, K, flush=True)
    gen = torch.Generator(device="cuda:0").manual_seed(M + N + K)
    packed = B.mnnq_pack_weights(torch.randn((N, K), generator=gen, device="cuda:0") * 0.02, mode=mode)
    x = torch.randn((M, K), generator=gen, device="cuda:0").half()
    q, s, z = (t.double() for t in B.mnnq_unpack_weights(packed, N, K, mode=mode))
    s, z, q = s[:, :, None], z[:, :, None], q.view(N, K // 64, 64)
    w = ((q - z) * s if mode == B.MODE_W4_ZP_INT else q * s + z).view(N, K)
    bias = torch.randn(N, generator=gen, device="cuda:0")
    exact = x.double() @ w.t() + bias.double()
    out = torch.full((M + 1, N), float("nan"), device="cuda:0")
    y = B.mnnq_linear_prefill_f16(packed, N, K, x, bias=bias, out=out[:M], mode=mode)
    assert torch.isnan(out[M]).all()                # nothing behind the last token
    assert (y.double() - exact).abs().max() <= 1e-5 * exact.abs().max()     # the layer's tolerance
    assert torch.equal(B.mnnq_linear_prefill_f16_o16(packed, N, K, x, bias=bias, mode=mode), y.half())
    if B.mnnq_plan_debug(5, M, N, K, mode)[0] == 0:     # a row factor changes neither the tile nor the order of the sums
        ones = torch.ones(M, device="cuda:0")
        assert torch.equal(B.mnnq_linear_prefill_f16(packed, N, K, x, row_scale=ones, bias=bias, mode=mode), y)


# One shape for each number of token blocks: nine waves (one block, sixteen waves on a CU) or five (eight) on a row tile, so that a CU
# holds one workgroup, and 515 row tiles: every workgroup walks over two, three of them over three.  33 and 17 chunks: waves with
# three and four of them, the last one half empty.
@pytest.mark.parametrize("M,K", [(5, 4160), (20, 2112), (40, 2112), (56, 2112)])
@pytest.mark.parametrize("form", list(FORMS))
def test_few_tokens_walk_over_row_tiles(form, M, K):
    mode, quant, linear = FORMS[form]
    if form.startswith("w8"):
        K = K // (2 if form == "w8planes" else 1) // 128 * 128 + 128
    N = 16 * 515
    print("few tokens, row tiles", form, M, N, K, flush=True)
    plan = B.mnnq_plan_debug(4, M, N, K, mode=mode)
    assert plan[0] == 1 and plan[4] // plan[3] == 1 and N // 16 > 2 * 256          # resident, one workgroup on each of 256 CUs
    W = synth.weights(N, K, 71 + M)
    xd = dev(synth.activations(M, K, 72 + M))
    bias = synth.weights(1, N, 73)[0] * 10
    q, s, z = quant(W)
    packed = B.mnnq_pack_weights(dev(W), mode=mode)
    xq, sx, _ = B.mnnq_quant_act(xd)
    y_o = linear(xq.cpu().numpy(), sx.cpu().numpy(), q, s, z, bias=bias, want_acc=False)[1]
    y = B.mnnq_linear_prefill(packed, N, K, xq, sx, bias=dev(bias), mode=mode)
    # fp32 sums of up to 68 group terms: the layer's tolerance, row tile by row tile
    err = np.abs(y.cpu().numpy() - y_o).reshape(M, 515, 16).max(axis=(0, 2))
    assert (err <= 1e-5 * np.abs(y_o).reshape(M, 515, 16).max(axis=(0, 2))).all()
    assert torch.equal(B.mnnq_linear_prefill_fused(packed, N, K, xd, bias=dev(bias), mode=mode), y)
