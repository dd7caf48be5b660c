"""Edges of the native calls' argument handling: what they refuse, what they accept and which errors they raise."""
import pytest
import torch

from paper_2506_10443_amd import binding as B

pytestmark = pytest.mark.gpu
N, K = 32, 128


@pytest.fixture(scope="module")
def packed():
    return B.mnnq_pack_weights(torch.randn(N, K, device="cuda:0"))


@pytest.mark.parametrize("call", [B.mnnq_linear_prefill_fused, B.mnnq_linear_prefill_fused_o16])
def test_an_empty_workspace_is_refused(packed, call):
    """A workspace that was given is the one that is used: an empty one is none (a null pointer), one too small is too small."""
    x = torch.randn(3, K, device="cuda:0")
    for size, status in ((0, -1), (16, -4)):
        with pytest.raises(B.MnnqError) as e:
            call(packed, N, K, x, workspace=torch.empty(size, dtype=torch.uint8, device="cuda:0"))
        assert e.value.status == status


def test_activations_with_trailing_dimensions(packed):
    """[M, K, 1] holds the rows of [M, K]; fewer than two dimensions are an IndexError, another K is a ValueError."""
    x = torch.randn(3, K, device="cuda:0")
    xq, sx, _ = B.mnnq_quant_act(x)
    calls = [(B.mnnq_linear_prefill_fused, x, ()), (B.mnnq_linear_prefill_fused_o16, x, ()),
             (B.mnnq_linear_prefill, xq, (sx,)), (B.mnnq_linear_prefill_o16, xq, (sx,)),
             (B.mnnq_linear_prefill_f16, x.half(), ()), (B.mnnq_linear_prefill_f16_o16, x.half(), ())]
    for call, a, rest in calls:
        y = call(packed, N, K, a, *rest)
        assert torch.equal(call(packed, N, K, a[:, :, None], *rest), y)
        with pytest.raises(IndexError):
            call(packed, N, K, a.view(-1), *rest)
        with pytest.raises(ValueError):
            call(packed, N, K, a.view(-1, K // 2), *rest)


def test_memory_that_torch_does_not_give(packed):
    """An output that the allocator refuses (here: for a limit set on this process) is torch's own error."""
    x = torch.randn(4096, K, device="cuda:0").half()
    torch.cuda.empty_cache()
    torch.cuda.set_per_process_memory_fraction(1e-6)
    try:
        with pytest.raises(torch.cuda.OutOfMemoryError):
            for _ in range(256):        # (whatever the allocator still holds runs out first)
                held = [B.mnnq_linear_prefill_f16(packed, N, K, x) for _ in range(256)]
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
    del x
    torch.cuda.synchronize()
