"""mnnq_pack_weights at the edges of its workgroups (32 rows, two or four chunks of 128 weights) and next to the ties of
its rounding, every packed form: codes and group parameters bit for bit the oracle's, and the buffer byte for byte the
one that mnnq_pack_from_quantized writes from them (padding included)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2506_10443_amd import binding as B, synth

pytestmark = pytest.mark.gpu
FORMS = {
    "w4": (B.MODE_W4_ZP_INT, oracle.quant_weights),
    "w4+plane": (B.MODE_W4_ZP_INT | B.WITH_MATRIX_PLANE, oracle.quant_weights),
    "w4min": (B.MODE_W4_MIN_FLOAT, oracle.quant_weights_minf),
    "w8": (B.MODE_W8_MIN_FLOAT | B.NATIVE_8BIT, oracle.quant_weights8),
    "w8planes": (B.MODE_W8_MIN_FLOAT, oracle.quant_weights8),
}


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def weights(N, K, levels, seed):
    """Random rows, constant and zero groups, groups of one sign, scales from 1e-36 to 1e36, and values on and one
    representable number beside the half steps of the quantizer."""
    rng = np.random.default_rng(seed)
    W = synth.weights(N, K, seed)
    g = W.reshape(N, K // 64, 64)
    for i in range(g.shape[0]):
        for j in range(g.shape[1]):
            kind = rng.integers(0, 8)
            if kind == 0:
                g[i, j] = np.float32(rng.choice([0.0, 0.25, -3.0]))
            elif kind == 1:
                g[i, j] = np.abs(g[i, j]) + np.float32(0.5)
            elif kind == 2:
                g[i, j] *= np.float32(10.0) ** np.float32(rng.integers(-34, 36))
            elif kind >= 5:
                half = (rng.integers(0, 2 * levels, 64) / np.float32(2.0)).astype(np.float32) * np.float32(2.0 ** -7)
                g[i, j] = half + np.float32(rng.integers(-4, 1)) * np.float32(2.0 ** -7)
                g[i, j] = np.nextafter(g[i, j], np.float32(rng.choice([-1.0, 1.0])), dtype=np.float32) if kind > 5 else g[i, j]
    return W


@pytest.mark.parametrize("N,K", [(16, 64), (16, 128), (48, 192), (32, 576), (272, 1088), (80, 1152), (4112, 256), (1040, 4096)])
@pytest.mark.parametrize("form", list(FORMS))
def test_pack_edges(form, N, K):
    mode, quant = FORMS[form]
    if form.startswith("w8") and K % 128:
        pytest.skip("int8 weights: K a multiple of 128")
    print("pack", form, N, K, flush=True)
    W = weights(N, K, 255 if form.startswith("w8") else 15, 5000 + N + K)
    q, s, z = quant(W)
    packed = torch.full((B.mnnq_packed_size(N, K, 64, mode),), 0xa5, dtype=torch.uint8, device="cuda:0")
    B.mnnq_pack_weights(dev(W), out=packed, mode=mode)
    qg, sg, zg = (t.cpu().numpy() for t in B.mnnq_unpack_weights(packed, N, K, mode=mode))
    assert np.array_equal(qg, q)
    assert np.array_equal(sg.view(np.uint32), s.view(np.uint32))
    assert np.array_equal(zg.view(np.uint8), np.ascontiguousarray(z).view(np.uint8))
    imported = torch.full_like(packed, 0x5a)
    B.mnnq_pack_from_quantized(dev(q), dev(s), dev(z), out=imported, mode=mode)
    assert torch.equal(packed, imported)
