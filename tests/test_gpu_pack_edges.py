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


def definition(W, levels, zero_point):
    """The quantizer's sequence of binary32 operations with the clamp min(max(c, 0), levels) of C (a NaN becomes 0)."""
    w = W.reshape(W.shape[0], -1, 64)
    with np.errstate(all="ignore"):
        mn, mx = np.fmin.reduce(w, axis=2), np.fmax.reduce(w, axis=2)
        if zero_point:
            mn, mx = np.fmin(mn, np.float32(0)), np.fmax(mx, np.float32(0))
        flat = mx == mn
        s = np.where(flat, np.float32(1), (mx - mn) / np.float32(levels))
        if zero_point:
            z = np.where(flat, np.float32(0), np.rint(-mn / s))
            c = np.rint(w / s[:, :, None]) + z[:, :, None]
            z = np.fmin(np.fmax(z, np.float32(0)), np.float32(255)).astype(np.uint8)
        else:
            z = mn
            c = np.rint((w - mn[:, :, None]) / s[:, :, None])
        q = np.where(flat[:, :, None], np.float32(0), np.fmin(np.fmax(c, np.float32(0)), np.float32(levels)))
    return q.astype(np.uint8).reshape(W.shape), s, z


@pytest.mark.parametrize("form", list(FORMS))
def test_pack_ends_of_the_range(form):
    """Groups whose range rounds to scale 0 (subnormal) or overflows, and groups with a NaN or an infinity among ordinary
    weights: codes and parameters of the definition."""
    mode = FORMS[form][0]
    levels = 255 if form.startswith("w8") else 15
    N, K = 48, 384
    print("pack ends", form, flush=True)
    W = synth.weights(N, K, 5500)
    g = W.reshape(N, K // 64, 64)
    tiny = np.float32(1.4e-45)
    rng = np.random.default_rng(5501)
    for i in range(N):
        kind = i % 12
        v = g[i, i % 6]
        if kind == 0:
            v[:] = tiny * rng.integers(0, 8, 64).astype(np.float32)           # scale 0, minimum 0
        elif kind == 1:
            v[:] = tiny * rng.integers(-3, 4, 64).astype(np.float32)          # scale 0, minimum below 0
        elif kind == 2:
            v[:] = tiny * rng.integers(-22, 23, 64).astype(np.float32)        # a scale of few units
        elif kind == 3:
            v[:] = np.float32(3e38) * rng.uniform(-1, 1, 64).astype(np.float32)
            v[:2] = np.float32(3e38), np.float32(-3e38)                       # the range overflows
        elif kind == 4:
            v[5] = np.nan
        elif kind == 5:
            v[rng.integers(0, 64, 20)] = np.nan
        elif kind == 6:
            v[:] = np.nan
        elif kind == 7:
            v[9] = np.inf
        elif kind == 8:
            v[63] = -np.inf
        elif kind == 9:
            v[0], v[1], v[2] = np.inf, -np.inf, np.nan
        elif kind == 10:
            v[:] = 0.0
            v[7] = np.nan
    q, s, z = definition(W, levels, mode & 15 == B.MODE_W4_ZP_INT)
    packed = B.mnnq_pack_weights(dev(W), mode=mode)
    qg, sg, zg = (t.cpu().numpy() for t in B.mnnq_unpack_weights(packed, N, K, mode=mode))
    bad = np.argwhere((qg != q).reshape(N, K // 64, 64).any(axis=2))
    assert bad.size == 0, [(int(n), int(n) % 12) for n, _ in bad]
    np.testing.assert_array_equal(sg, s)            # (NaN equals NaN)
    np.testing.assert_array_equal(zg, z)
