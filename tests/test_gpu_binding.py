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
