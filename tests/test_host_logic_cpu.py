"""Host logic of the launchers, checked without a GPU through mnnq_plan_debug: for every layer shape of
the benchmark models the chosen kernel configuration fits the hardware limits the kernels assume
(1024 threads, 160 KiB of LDS per workgroup), covers the whole
problem, and is the one the design documents for the Qwen2-7B shapes.  Nothing is launched."""
import os

import pytest

from paper_2506_10443_amd import binding as B, synth

LDS_GEMM, LDS_GEMV = 160 * 1024, 160 * 1024


@pytest.fixture(scope="module", autouse=True)
def built():
    if not os.path.exists(B.LIB_PATH):
        import __graft_entry__
        __graft_entry__.build()
    for v in ("MNNQ_PREFILL_TILE", "MNNQ_DECODE_KSPLIT", "MNNQ_DECODE_WAVES", "MNNQ_DECODE_EARLY", "MNNQ_W8_PLANES"):
        B.mnnq_debug_set(v, None)


def shapes():
    out = []
    for model, spec in synth.MODELS.items():
        for fused in (True, False):
            for name, N, K in synth.block_layers(model, fused=fused):
                out.append((model, name, spec["prefill_m"], N, K))
        if spec["lm_head"]:
            out.append((model, "lm_head", spec["prefill_m"], *spec["lm_head"]))
    return out


@pytest.mark.parametrize("mode", [B.MODE_W4_ZP_INT, B.MODE_W4_MIN_FLOAT, B.MODE_W8_MIN_FLOAT])
@pytest.mark.parametrize("model,name,M,N,K", shapes())
def test_prefill_plan_fits_and_covers(model, name, M, N, K, mode):
    for m in sorted({M, 17, 100, 129, 300}):
        bm, bn, ks, s, waves, lds, wgs, merged = B.mnnq_plan_debug(0, m, N, K, mode)
        assert (bm, bn) in ((64, 64), (64, 128), (128, 128), (256, 128), (128, 256), (128, 192)) and ks in (1, 2, 4) and s in (1, 2)
        assert (bm == 64) == (m <= 128 and not merged and not (m > 64 and -(-N // 128) >= 1024))
        assert ks < 4 or bm == 64
        assert waves in (4, 8, 16) and waves * 64 <= 1024 and waves % ks == 0
        assert lds <= LDS_GEMM
        if waves // ks == 4:
            assert 2 * lds <= LDS_GEMM or ks >= 2      # the four-wave forms count on two workgroups per CU
        assert wgs >= -(-m // bm) * s * -(-N // bn)     # every output tile (and K part) has a workgroup
        assert merged == (1 if mode == B.MODE_W8_MIN_FLOAT else 0)
        if merged:
            assert bm == 128


@pytest.mark.parametrize("mode", [B.MODE_W4_ZP_INT, B.MODE_W4_MIN_FLOAT, B.MODE_W8_MIN_FLOAT])
@pytest.mark.parametrize("model,name,M,N,K", shapes())
def test_decode_plan_fits_and_covers(model, name, M, N, K, mode):
    chunks = -(-(K * (2 if mode == B.MODE_W8_MIN_FLOAT else 1)) // 128)
    tiles = N // 16
    for what in (1, 2):
        if chunks * 128 > 126976:
            with pytest.raises(B.MnnqError):
                B.mnnq_plan_debug(what, 1, N, K, mode)
            continue
        waves, ks, unroll, prefetch, lds, wgs, tiles_per_wg, _ = B.mnnq_plan_debug(what, 1, N, K, mode)
        assert waves in (4, 8, 16) and ks in (1, 2, 4, 8, 16) and waves % ks == 0 and tiles_per_wg == waves // ks
        assert lds <= LDS_GEMV
        assert wgs * tiles_per_wg >= tiles
        per_wave = -(-chunks // ks)
        assert prefetch == (1 if per_wave > unroll else 0)      # else the whole range sits in registers


def test_documented_plans_of_the_qwen2_7b_block():
    # (the tiled GEMM's; without the plane the call runs the K-split kernel for all but gate|up)
    assert [B.mnnq_plan_debug(4, 1024, n, k)[0] for n, k in ((37888, 3584), (4608, 3584), (3584, 3584), (3584, 18944))] == [0, 3, 3, 3]
    plan = lambda n, k: B.mnnq_plan_debug(0, 1024, n, k)[:5]
    assert plan(37888, 3584) == [256, 128, 1, 1, 8]      # gate|up: two workgroups of eight waves per CU
    assert plan(4608, 3584) == [128, 192, 2, 1, 8]       # q|k|v: two K parts of four waves
    assert plan(3584, 3584) == [128, 128, 2, 1, 16]      # o
    assert plan(3584, 18944) == [128, 128, 2, 1, 16]     # down
    assert B.mnnq_plan_debug(1, 1, 37888, 3584)[:4] == [4, 4, 7, 0]      # GEMV: four waves per row tile, 7 chunks each
    assert B.mnnq_plan_debug(1, 1, 3584, 18944)[:4] == [16, 16, 12, 0]   # 148 chunks over sixteen waves
    assert B.mnnq_plan_debug(1, 1, 4096, 14336)[:4] == [16, 16, 7, 0]    # (Llama-3-8B down) 112 chunks: seven each
    assert B.mnnq_plan_debug(2, 1, 4608, 3584)[0] == 8                    # fused quantizer: larger workgroups
    # the activation row is handled under the weight stream where (nearly) every wave's registers are filled:
    # small layers with at most two chunks fewer per wave than registers for them, and exactly fitting ones
    early = lambda what, n, k: B.mnnq_plan_debug(what, 1, n, k)[7]
    shapes = ((4608, 3584), (3584, 3584), (3584, 18944), (37888, 3584))
    assert [early(1, n, k) for n, k in shapes] == [1, 1, 0, 1]
    assert [early(2, n, k) for n, k in shapes] == [1, 1, 0, 1]
    assert B.mnnq_plan_debug(2, 1, 3584, 3584)[:3] == [8, 8, 4]    # fused o: eight waves per row tile, 3 - 4 chunks each
    assert early(1, 1536, 8960) == 0 and early(1, 2048, 1536) == 1  # Qwen2-1.5B down (4 - 5 of 8 chunks) and q|k|v


def test_plans_of_the_byte_form_of_int8_weights():
    """mode MNNQ_W8_MIN_FLOAT | MNNQ_NATIVE_8BIT: the GEMV keeps seven chunks of two kilobytes per wave in
    registers (a rolling window beyond sixteen waves per row tile), the GEMM runs tiles of 128 tokens."""
    NB = B.MODE_W8_MIN_FLOAT | B.NATIVE_8BIT
    for model, name, M, N, K in shapes():
        if K % 128:
            continue
        chunks = K // 128
        for what in (1, 2):
            waves, ks, unroll, prefetch, lds, wgs, tiles_per_wg, early = B.mnnq_plan_debug(what, 1, N, K, NB)
            assert unroll == 7 and early == 0 and waves % ks == 0 and tiles_per_wg == waves // ks
            assert ks == 16 or -(-chunks // ks) <= 7
            assert prefetch == (1 if -(-chunks // ks) > 7 else 0)
            assert (waves, ks) in (((4, 1), (4, 2), (4, 4), (8, 8), (16, 16)) if what == 1 else
                                   ((8, 1), (8, 2), (8, 4), (8, 8), (16, 16)))
            assert lds <= LDS_GEMV and wgs * tiles_per_wg >= N // 16
        bm, bn, kparts, s, w, lds, wgs, form = B.mnnq_plan_debug(0, M, N, K, NB)
        assert bm == 128 and bn in (128, 192, 256) and form == 2 and kparts in (1, 2) and lds <= LDS_GEMM
        assert bn == 128 or w == 4 * kparts         # (the wide tiles: four waves of 16 tokens x bn / 4 columns per part)
        assert wgs >= -(-M // 128) * s * -(-N // bn)
    assert B.mnnq_plan_debug(1, 1, 152064, 3584, NB)[:4] == [4, 4, 7, 0]     # LM head: 28 chunks on four waves
    assert B.mnnq_plan_debug(1, 1, 3584, 18944, NB)[:4] == [16, 16, 7, 1]    # down: 148 chunks, a window of seven


@pytest.mark.parametrize("mode", [B.MODE_W4_ZP_INT, B.MODE_W4_MIN_FLOAT, B.MODE_W8_MIN_FLOAT, B.MODE_W8_MIN_FLOAT | B.NATIVE_8BIT])
def test_both_plan_views_show_the_tiled_kernel_that_runs(mode):
    """Where the fused call takes the tiled GEMM, what = 4 and what = 0 name the same tile, waves and workgroups, and a forced
    tile is what both show; every tile and K split is seen."""
    seen = set()
    for m in (65, 129, 200, 333, 512, 1024, 2048):
        for n, k in ((37888, 3584), (28672, 4096), (17920, 1536), (6144, 4096), (4608, 3584), (4096, 14336), (11264, 1536), (32768, 1536), (152064, 3584)):
            family, bm, bn, waves, _, _, groups, _ = B.mnnq_plan_debug(4, m, n, k, mode)
            t = B.mnnq_plan_debug(0, m, n, k, mode)
            assert t[5] <= LDS_GEMM and t[6] >= -(-m // t[0]) * t[3] * -(-n // t[1])
            seen.add(tuple(t[:3]))
            if family == 0:
                assert (bm, bn, waves, groups) == (t[0], t[1], t[4], t[6])
    if mode in (B.MODE_W4_ZP_INT, B.MODE_W8_MIN_FLOAT | B.NATIVE_8BIT):
        assert {(128, 256, 1), (128, 192, 1), (128, 256, 2), (128, 192, 2)} <= seen
        try:
            for tile, columns, parts in (("x1", 256, 1), ("x1k", 256, 2), ("c1", 192, 1), ("c1k", 192, 2)):
                B.mnnq_debug_set("MNNQ_PREFILL_TILE", tile)
                assert B.mnnq_plan_debug(0, 1024, 37888, 3584, mode)[:5] == [128, columns, parts, 1, 4 * parts]
                assert B.mnnq_plan_debug(4, 1024, 37888, 3584, mode)[:4] == [0, 128, columns, 4 * parts]
        finally:
            B.mnnq_debug_set("MNNQ_PREFILL_TILE", None)


def test_documented_plans_for_few_tokens():
    """The tiled GEMM for 17 .. 128 tokens: 64-row tiles, 64 columns wide unless there are very many,
    the K range in more parts the fewer workgroups there are; very many tiles beyond 64 tokens take
    128-row tiles.  (Few tokens have kernels of their own, and few tiles the K-split one: it runs in this
    range for short rows of many columns, or where those are switched off.)"""
    assert B.mnnq_plan_debug(4, 128, 32768, 1536)[0] == 0 and B.mnnq_plan_debug(4, 64, 3584, 18944)[0] == 2
    plan = lambda m, n, k: B.mnnq_plan_debug(0, m, n, k)[:5]
    assert plan(64, 4608, 3584) == [64, 64, 4, 1, 16]        # q|k|v: 72 workgroups
    assert plan(64, 3584, 18944) == [64, 64, 4, 2, 16]       # down: long rows cut in two as well
    assert plan(64, 37888, 3584) == [64, 64, 2, 1, 8]        # gate|up: 592 workgroups, two to three per CU
    assert plan(128, 37888, 3584) == [64, 64, 1, 1, 4]       # 1184 workgroups of four waves
    assert plan(64, 152064, 3584) == [64, 128, 1, 1, 4]      # lm_head: 1188 tiles of 64 x 128
    assert plan(128, 152064, 3584) == [128, 128, 1, 1, 4]    # ... and 128-row tiles beyond 64 tokens


def test_switches_and_errors():
    B.mnnq_debug_set("MNNQ_PREFILL_TILE", "s1")
    try:
        assert B.mnnq_plan_debug(0, 1024, 37888, 3584)[:5] == [128, 128, 1, 1, 4]
    finally:
        B.mnnq_debug_set("MNNQ_PREFILL_TILE", None)
    B.mnnq_debug_set("MNNQ_W8_PLANES", "1")
    try:
        assert B.mnnq_plan_debug(0, 1024, 37888, 3584, B.MODE_W8_MIN_FLOAT)[7] == 0
    finally:
        B.mnnq_debug_set("MNNQ_W8_PLANES", None)
    # the library does not read the environment: a stray variable changes nothing
    os.environ["MNNQ_PREFILL_TILE"] = "s1"
    try:
        assert B.mnnq_plan_debug(0, 1024, 37888, 3584)[:5] != [128, 128, 1, 1, 4]
    finally:
        os.environ.pop("MNNQ_PREFILL_TILE")
    L = B.lib()
    assert L.mnnq_debug_set(b"MNNQ_NO_SUCH_SWITCH", b"1") == -3 and L.mnnq_debug_set(None, b"1") == -1
    assert L.mnnq_debug_set(b"MNNQ_PREFILL_TILE", b"0123456789abcdef") == -4
    assert L.mnnq_plan_debug(0, 4, 16, 128, 64, 0, None) == -1
    import ctypes
    out = (ctypes.c_int32 * 8)()
    p = ctypes.cast(out, ctypes.c_void_p)
    assert L.mnnq_plan_debug(3, 4, 16, 128, 64, 0, p) == -3
    assert L.mnnq_plan_debug(0, 0, 16, 128, 64, 0, p) == -2
    assert L.mnnq_plan_debug(1, 1, 16, 100, 64, 0, p) == -2
    assert L.mnnq_plan_debug(1, 1, 16, 131072, 64, 0, p) == -3    # longer than the GEMV stages in LDS
    assert L.mnnq_plan_debug(1, 1, 16, 53248, 64, 0, p) == 0 and out[4] > 64 * 1024 and out[4] <= 160 * 1024


@pytest.mark.parametrize("what,mode", [(4, B.MODE_W4_ZP_INT), (4, B.MODE_W4_MIN_FLOAT), (4, B.MODE_W8_MIN_FLOAT),
                                       (4, B.MODE_W8_MIN_FLOAT | B.NATIVE_8BIT), (5, B.MODE_W4_ZP_INT),
                                       (5, B.MODE_W4_MIN_FLOAT), (5, B.MODE_W8_MIN_FLOAT)])
def test_few_token_kernels_run_with_the_waves_they_are_built_for(what, mode):
    """No split of K, a forced one among them, launches more waves than the chosen kernel's registers allow."""
    try:
        for force in (None, 1, 2, 4, 8, 16):
            B.mnnq_debug_set("MNNQ_DECODE_KSPLIT", force)
            for m in (2, 16, 17, 33, 49, 64):
                for n, k in ((1536, 1536), (4608, 3584), (3584, 18944), (28672, 4096), (48, 128)):
                    family, tokens, rows, waves, most, held = B.mnnq_plan_debug(what, m, n, k, mode)[:6]
                    assert 1 <= waves <= most or family == 0
                    if family == 1:     # every chunk of the packed row in a wave's registers
                        chunks = -(-k // 128) * (2 if mode == B.MODE_W8_MIN_FLOAT else 1)
                        assert -(-chunks // waves) <= held
    finally:
        B.mnnq_debug_set("MNNQ_DECODE_KSPLIT", None)


@pytest.mark.parametrize("mode", [B.MODE_W4_ZP_INT, B.MODE_W4_MIN_FLOAT, B.MODE_W8_MIN_FLOAT, B.MODE_W8_MIN_FLOAT | B.NATIVE_8BIT])
def test_few_tokens_of_long_rows_share_a_tile_among_few_waves(mode):
    """One block of tokens, rows too long for the registers: four waves on a row tile, eight where tiles are few."""
    for n, k, waves in ((4096, 14336, 4), (3584, 18944, 4), (2048, 8448, 4), (2032, 8448, 8), (1536, 8960, 8)):
        for m in (2, 16):
            assert B.mnnq_plan_debug(4, m, n, k, mode)[:4] == [2, 16, 16, waves]
    assert B.mnnq_plan_debug(4, 17, 4096, 14336, mode)[3] == 8
    # rows that would fit the registers of more than eight waves, one tile per workgroup; with a second tile they stay there
    plane8 = mode == B.MODE_W8_MIN_FLOAT
    for n, k, waves in ((4096, 8192, 4), (3584, 6784, 4), (1536, 6784, 8)) if not plane8 else ((4096, 4096, 4), (1008, 3840, 8)):
        assert B.mnnq_plan_debug(4, 2, n, k, mode)[:4] == [2, 16, 16, waves]
    for n, k in ((4608, 8192), (4096, 4096), (4096, 3584)) if not plane8 else ((4608, 4096), (4096, 2048)):
        assert B.mnnq_plan_debug(4, 2, n, k, mode)[0] == 1


def test_few_token_kernels_where_they_are_the_faster_ones():
    """Which layers leave the few-token kernels below 64 tokens, and which stay with them beyond: the shapes measured on
    both sides of each line."""
    few = lambda m, n, k, mode=B.MODE_W4_ZP_INT: B.mnnq_plan_debug(4, m, n, k, mode)[0] in (1, 2)
    planes = B.MODE_W8_MIN_FLOAT
    for mode in (B.MODE_W4_ZP_INT, B.MODE_W4_MIN_FLOAT, B.MODE_W4_ZP_INT | B.WITH_MATRIX_PLANE, planes | B.NATIVE_8BIT):
        assert all(few(16, n, k, mode) for n, k in ((13824, 5120), (37888, 3584)))
        # both operands streamed: one round of workgroups and more
        assert few(64, 4096, 14336, mode) and not few(17, 5120, 5120, mode) and not few(64, 13824, 5120, mode)
        # two slices of tokens: one round and more
        assert few(128, 2048, 1536, mode) and not few(65, 2560, 2560, mode) and not few(128, 3584, 3584, mode)
        assert few(48, 37888, 3584, mode)
    # 49 tokens and more: three or five waves for a row leave much of a CU empty; with the plane always
    assert few(64, 20480, 2048) and few(64, 28672, 4096) and few(64, 37888, 3584) and few(64, 28672, 4096, planes | B.NATIVE_8BIT)
    assert not few(49, 28672, 1152) and not few(49, 28672, 2560) and few(64, 20480, 2560)
    assert all(few(m, n, k, B.MODE_W4_ZP_INT | B.WITH_MATRIX_PLANE) for m in (49, 64) for n, k in ((37888, 3584), (40960, 2304)))
    assert few(64, 8192, 2048, B.MODE_W4_MIN_FLOAT) and not few(49, 14336, 4096, B.MODE_W4_MIN_FLOAT)
    # int8 nibble planes: twice the chunks, against the tiled GEMM that merges them
    assert few(48, 8192, 8192, planes) and few(32, 13824, 5120, planes) and not few(48, 13824, 5120, planes)
    assert not any(few(m, n, k, planes) for m in (17, 33, 64) for n, k in ((28672, 4096), (37888, 3584)))
    assert few(128, 2560, 2560, planes)


@pytest.mark.parametrize("what,mode,family", [(5, B.MODE_W4_ZP_INT, 0), (5, B.MODE_W4_ZP_INT, 3), (5, B.MODE_W8_MIN_FLOAT, 3),
                                              (4, B.MODE_W4_MIN_FLOAT, 3), (4, B.MODE_W4_ZP_INT | B.WITH_MATRIX_PLANE, 7)])
def test_tiles_are_dealt_evenly_to_the_xcds(what, mode, family):
    """Columns of tiles that are no multiple of the eight XCDs: no more workgroups than tiles rounded up to eight (one set of
    whole columns per XCD was up to 40 of 28 columns), since the rules of the dispatch count tiles per CU."""
    met = 0
    for m in (129, 333, 802, 1290, 1792):
        for n, k in ((4608, 3584), (2560, 6400), (1136, 3712), (1040, 2688), (3440, 10496)):
            f, tokens, rows, _, _, _, groups, _ = B.mnnq_plan_debug(what, m, n, k, mode)
            if f == family:
                met += 1
                tiles = -(-m // tokens) * -(-n // rows)
                assert tiles <= groups < tiles + 8
    assert met


def test_k_split_int8_gemm_where_its_rounds_cost_less():
    """Shapes measured on both sides of the line to the tiled GEMM: full rounds of many columns and short rows are the tiled
    one's; long rows, and columns that the tiled GEMM deals unevenly to the XCDs, the K-split one's."""
    ksplit = lambda m, n, k, mode=B.MODE_W4_ZP_INT: B.mnnq_plan_debug(4, m, n, k, mode)[0] == 3
    w8 = B.MODE_W8_MIN_FLOAT | B.NATIVE_8BIT
    assert not any(ksplit(m, n, k, w8) for m, n, k in ((113, 28672, 4096), (256, 28672, 4096), (377, 17920, 1536), (1617, 4096, 4096)))
    assert not any(ksplit(m, n, k) for m, n, k in ((256, 15952, 1664), (356, 15952, 1664), (707, 5104, 1408)))
    assert all(ksplit(m, n, k, w8) for m, n, k in ((784, 4096, 14336), (771, 4608, 3584), (529, 4000, 12672), (333, 4096, 4096)))
    assert all(ksplit(m, n, k) for m, n, k in ((1125, 3584, 3584), (803, 4608, 3584), (1181, 4096, 14336), (333, 4096, 4096)))


def test_int8_tiles_that_the_shapes_were_measured_fastest_on():
    """Shapes at which one kernel beat the others by 3 % and more, on rows and fused: the K-split kernel (3), and of the tiled
    GEMM's forms (tokens, columns, waves)."""
    w8 = B.MODE_W8_MIN_FLOAT | B.NATIVE_8BIT
    plan = lambda m, n, k, mode: tuple(B.mnnq_plan_debug(4, m, n, k, mode)[:4])
    low = B.MODE_W4_MIN_FLOAT
    # float minima of 4-bit codes: 128 x 128 of four waves, 10 - 20 % ahead of the K-split kernel ...
    for m, n, k in ((2048, 6144, 4096), (427, 24288, 3456), (1803, 5824, 3840), (512, 17920, 1536), (333, 28672, 4096), (1914, 5856, 3200)):
        assert plan(m, n, k, low) == (0, 128, 128, 4)
    # ... and behind it
    for m, n, k in ((147, 16672, 1792), (502, 8224, 2048), (1963, 2544, 6144), (467, 9840, 2432), (391, 16880, 3072)):
        assert plan(m, n, k, low)[0] == 3
    for m, n, k in ((1024, 37888, 3584), (2048, 28672, 4096), (932, 37280, 3840), (924, 23456, 1280), (1974, 10688, 1280)):
        assert plan(m, n, k, B.MODE_W4_ZP_INT) == (0, 256, 128, 8)
    for m, n, k in ((225, 28160, 1792), (428, 15184, 1664)):
        assert plan(m, n, k, B.MODE_W4_ZP_INT) == (0, 128, 128, 8)
    for m, n, k in ((634, 31168, 1664), (1220, 14720, 3456)):
        assert plan(m, n, k, w8) == (0, 128, 128, 8)
    assert plan(1024, 37888, 3584, w8) == (0, 128, 256, 4) and plan(2048, 6144, 4096, w8) == (0, 128, 192, 4)


def test_fp16_activations_of_17_to_64_tokens_take_the_faster_kernel():
    """Shapes at which the few-token kernel (families 1, 2) or the K-split one (3) was measured 7 % and more ahead."""
    plan = lambda m, n, k, mode: B.mnnq_plan_debug(5, m, n, k, mode)[0]
    for m, n, k in ((56, 19264, 1664), (58, 21632, 1920), (59, 17360, 1536), (43, 19536, 1664), (25, 4016, 2176), (24, 16448, 4096), (18, 4000, 1408)):
        assert plan(m, n, k, B.MODE_W4_ZP_INT) in (1, 2)
    for m, n, k in ((32, 14432, 1792), (24, 5824, 1792), (46, 1008, 1792), (62, 1296, 1024), (32, 7040, 1984), (64, 1328, 17024)):
        assert plan(m, n, k, B.MODE_W4_ZP_INT) == 3
    for m, n, k in ((54, 10480, 1088), (53, 9152, 1664), (24, 36224, 3840), (23, 992, 1280), (36, 1040, 1280), (48, 18608, 1280)):
        assert plan(m, n, k, B.MODE_W4_MIN_FLOAT) in (1, 2)
    # rows too long for the registers: the first tokens of a second block, whose 16-row tiles are nearly empty
    for m, n, k, mode in ((17, 3600, 11776, B.MODE_W4_MIN_FLOAT), (18, 3584, 15616, B.MODE_W4_MIN_FLOAT), (18, 2064, 13568, B.MODE_W8_MIN_FLOAT)):
        assert plan(m, n, k, mode) == 2 and plan(m + 6, n, k, mode) == 3 and plan(m, n + 4096, k, mode) == 3
    for m, n, k in ((42, 31888, 1152), (42, 2416, 2048), (20, 14736, 2688), (49, 1616, 1536), (64, 1760, 8320)):
        assert plan(m, n, k, B.MODE_W4_MIN_FLOAT) == 3
