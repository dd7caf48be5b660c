"""The fused one-token call on both sides of the lines of its rule: quantizer in every workgroup, or once in front."""
import pytest
import torch

from paper_2506_10443_amd import binding as B
from paper_2506_10443_amd import synth

pytestmark = pytest.mark.gpu
W8N = B.MODE_W8_MIN_FLOAT | B.NATIVE_8BIT

# sixteen waves per row tile: one round of workgroups and one more tile (256 CUs), very long rows too; the 64 MiB line of int4 weights
# (48 for eight waves); int8 bytes stay in one kernel beyond it, and so do waves whose registers are exactly filled: up to 96 MiB, and
# at every size where a CU holds three workgroups of the kernel (28 chunks and zero points), not where it holds two
ROUTES = [(4096, 8320, B.MODE_W4_ZP_INT, False), (4112, 8320, B.MODE_W4_ZP_INT, True), (4096, 7296, W8N, False), (4112, 7296, W8N, True),
          (4112, 14464, W8N, True), (33024, 1856, B.MODE_W4_ZP_INT, False), (62000, 1856, B.MODE_W4_ZP_INT, True),
          (62000, 1856, B.MODE_W4_MIN_FLOAT, True), (8192, 8064, B.MODE_W4_ZP_INT, False), (16384, 6080, B.MODE_W4_ZP_INT, True), (21504, 3584, B.MODE_W4_MIN_FLOAT, False), (52000, 3584, B.MODE_W4_ZP_INT, False),
          (38000, 3072, W8N, False), (52000, 3520, B.MODE_W4_ZP_INT, False), (52000, 3584, B.MODE_W4_MIN_FLOAT, True),
          (48000, 4096, B.MODE_W4_ZP_INT, True), (40000, 4096, B.MODE_W4_ZP_INT, False), (1024, 65536, B.MODE_W4_MIN_FLOAT, False)]


@pytest.mark.parametrize("N,K,mode,two", ROUTES)
def test_fused_decode_route(N, K, mode, two):
    print("fused decode route", N, K, mode, flush=True)
    x = torch.from_numpy(synth.activations(1, K, 5)).cuda()
    gen = torch.Generator(device="cuda").manual_seed(7)
    packed = B.mnnq_pack_weights(torch.randn((N, K), generator=gen, device="cuda").mul_(0.02), mode=mode)
    xq, sx, _ = B.mnnq_quant_act(x)
    want = B.mnnq_linear_decode(packed, N, K, xq[0].contiguous(), sx, mode=mode)
    ws = torch.zeros(B.mnnq_workspace_size(1, N, K, 64, mode), dtype=torch.uint8, device="cuda")
    out = B.mnnq_linear_decode_fused(packed, N, K, x[0].contiguous(), workspace=ws, mode=mode)
    # the codes are in the workspace if, and only if, the quantizer ran on its own
    assert torch.equal(ws[:K].view(torch.int8), xq[0] if two else torch.zeros_like(xq[0]))
    # the same codes, the same waves per row tile and the same order of the sums: bits, on the route that was taken and on the other
    assert torch.equal(out, want)
    B.mnnq_debug_set("MNNQ_FUSED_TWO_KERNEL_MIB", 100000 if two else 0)
    try:
        ws.zero_()
        other = B.mnnq_linear_decode_fused(packed, N, K, x[0].contiguous(), workspace=ws, mode=mode)
        assert torch.equal(ws[:K].view(torch.int8), torch.zeros_like(xq[0]) if two else xq[0])
    finally:
        B.mnnq_debug_set("MNNQ_FUSED_TWO_KERNEL_MIB", None)
    assert torch.equal(other, want)


@pytest.mark.parametrize("K", [8256, 10240, 10304, 12288, 12352, 14272, 14336, 16384, 16448, 20480, 20544, 24576, 24640])
@pytest.mark.parametrize("mode", [B.MODE_W4_ZP_INT, B.MODE_W4_MIN_FLOAT, B.MODE_W8_MIN_FLOAT])
def test_long_rows_quantized_under_the_weight_stream(mode, K):
    """Sixteen waves per row tile: around the numbers of chunks a wave holds (5 to 10, then 12, then a window), waves with one chunk
    fewer, odd numbers of groups, the last row tile alone in its workgroup.  Int8 nibble planes run over half the columns twice."""
    if mode == B.MODE_W8_MIN_FLOAT:
        K = K // 2 // 128 * 128
    N = 48
    print("long rows", K, mode, flush=True)
    x = torch.from_numpy(synth.activations(1, K, 11)).cuda()
    x[0, K - 1] = 500.0                             # the row's maximum is its last value
    gen = torch.Generator(device="cuda").manual_seed(K)
    packed = B.mnnq_pack_weights(torch.randn((N, K), generator=gen, device="cuda").mul_(0.02), mode=mode)
    xq, sx, _ = B.mnnq_quant_act(x)
    assert abs(float(sx[0]) - 500.0 / 127) < 1e-5
    guard = torch.full((N + 1,), 7.5, device="cuda")
    out = B.mnnq_linear_decode_fused(packed, N, K, x[0].contiguous(), mode=mode, out=guard[:N])
    # the same codes and the same order of the sums as quantizer and layer one after the other
    assert torch.equal(out, B.mnnq_linear_decode(packed, N, K, xq[0].contiguous(), sx, mode=mode))
    assert float(guard[N]) == 7.5
    zero = B.mnnq_linear_decode_fused(packed, N, K, torch.zeros(K, device="cuda"), mode=mode)
    assert bool((zero == 0).all())


@pytest.mark.parametrize("K", [8256, 10304, 12288, 12352, 14336, 16384, 16448, 20480, 20544, 24640])
@pytest.mark.parametrize("mode", [B.MODE_W4_ZP_INT, B.MODE_W4_MIN_FLOAT, B.MODE_W8_MIN_FLOAT])
def test_long_fp16_rows_staged_under_the_weight_stream(mode, K):
    """The same with fp16 activations: the form that requests the row ahead of the weights against the one behind branches (the same
    waves and order of the sums: bits), and against the kernel of two tokens."""
    if mode == B.MODE_W8_MIN_FLOAT:
        K = K // 2 // 128 * 128
    N = 48
    print("long fp16 rows", K, mode, flush=True)
    x = torch.from_numpy(synth.activations(1, K, 13)).cuda().half()
    gen = torch.Generator(device="cuda").manual_seed(K)
    packed = B.mnnq_pack_weights(torch.randn((N, K), generator=gen, device="cuda").mul_(0.02), mode=mode)
    guard = torch.full((N + 1,), 7.5, device="cuda")
    out = B.mnnq_linear_decode_f16(packed, N, K, x[0].contiguous(), mode=mode, out=guard[:N])
    assert float(guard[N]) == 7.5
    B.mnnq_debug_set("MNNQ_DECODE_EARLY", 0)
    try:
        other = B.mnnq_linear_decode_f16(packed, N, K, x[0].contiguous(), mode=mode)
    finally:
        B.mnnq_debug_set("MNNQ_DECODE_EARLY", None)
    assert torch.equal(out, other)
    two = B.mnnq_linear_prefill_f16(packed, N, K, torch.cat([x, x]), mode=mode)
    # fp32 sums of up to 386 group terms in another order
    assert float((two[0] - out).abs().max()) <= 1e-5 * float(two.abs().max())
