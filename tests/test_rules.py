"""The rules that choose kernels, on the CPU."""
import ctypes
import math

import numpy as np
import pytest

import rules
import synth
from oracle import xcache_oracle as xo

UNIT = math.log2(math.e)  # of a score bound per sqrt(d), besides its 2%


def _bound(gq, gk, rope=0):
    gq, gk = (np.asarray(g, np.float32) for g in (gq, gk))
    return rules.lib().score_bound(gq, gk, len(gq), rope)


@pytest.mark.parametrize("d", [64, 128])
def test_score_bound_of_the_gains(d):
    one = 1.02 * math.sqrt(d) * UNIT
    assert _bound(np.full(d, 1.5), np.full(d, -2.0)) == pytest.approx(3 * one, rel=1e-6)
    # products of 1 in every dimension, but a rotation mixes the two of a pair
    gq, gk = np.tile([4.0, 0.25], d // 2), np.tile([0.25, 4.0], d // 2)
    assert _bound(gq, gk) == pytest.approx(one, rel=1e-6)
    assert _bound(gq, gk, rope=1) == pytest.approx(16 * one, rel=1e-6)
    # one dimension, one pair
    gq, gk = np.ones(d), np.ones(d)
    gq[d - 1], gk[d - 2] = 3.0, 5.0
    assert _bound(gq, gk) == pytest.approx(5 * one, rel=1e-6)
    assert _bound(gq, gk, rope=1) == pytest.approx(15 * one, rel=1e-6)
    for bad in (math.inf, -math.inf, math.nan):
        gq[d // 2] = bad
        for g in ((gq, gk), (gk, gq)):
            for rope in (0, 1):
                assert _bound(*g, rope) == math.inf
    assert _bound(np.full(d, 1e30), np.full(d, 1e30)) == math.inf


def test_bounded_attention_rule():
    b = rules.lib().bounded
    assert b(64.0, 1.0, 1) and not b(np.nextafter(np.float32(64), np.float32(65)), 1.0, 1)
    # score + log2(keys) + log2(values) up to 120
    assert b(50.0, 2.0 ** 50, 1 << 20) and not b(50.0, 2.0 ** 50.01, 1 << 20) and not b(50.0, 2.0 ** 50, (1 << 20) + 9999)
    assert b(16.6, 2.0 ** 79, 1 << 24)
    # score - log2(values) up to 92
    assert b(50.0, 2.0 ** -42, 64) and not b(50.0, 2.0 ** -42.01, 64) and not b(16.6, 0.0, 64)
    for bad in (math.inf, math.nan):
        assert not b(bad, 1.0, 64) and not b(16.6, bad, 64)


def test_attention_wide_waves():
    """64-query waves wherever they measured faster (queries, keys, head dim, items on 256 CUs)."""
    wide = rules.lib().wide_waves
    for case in ((9522, 64, 128, 570), (9522, 129, 128, 570), (9522, 21060, 128, 570), (3510, 256, 128, 84), (160, 64, 64, 8),
                 (7020, 128, 64, 448), (3245, 6490, 64, 208), (129, 129, 128, 2)):
        assert wide(*case, 256), case
    for case in ((33, 448, 64, 8), (128, 1024, 128, 8), (128, 128, 64, 512), (9522, 128, 128, 570), (9522, 65, 128, 570),
                 (3245, 128, 64, 208), (3245, 65, 64, 256)):
        assert not wide(*case, 256), case


def test_attention_splits():
    """Split wherever a split measured faster, whole where it did not ((items, key tiles) on 256 CUs), and never past what the
    workspace holds."""
    n = rules.lib().splits
    for case in ((16, 8), (36, 8), (36, 9), (48, 10), (64, 9), (64, 12), (112, 14), (128, 16), (336, 330), (24, 48), (4, 10)):
        assert n(*case, 256, 1 << 40) > 1, case
    for case in ((1, 7), (16, 7), (48, 7), (84, 8), (112, 10), (128, 10), (208, 102), (256, 64), (570, 32)):
        assert n(*case, 256, 1 << 40) == 1, case
    for items in (1, 4, 24, 60, 336):
        for tiles in (1, 7, 8, 10, 33, 330):
            free = n(items, tiles, 256, 1 << 40)
            assert 1 <= free <= max(1, min(16, tiles // 2))
            for most in range(0, 18):
                assert n(items, tiles, 256, most) <= max(most, 1)
            assert n(items, tiles, 256, free) == free


@pytest.mark.parametrize("action", [0.5, 40.0])
def test_value_bounds_hold(action):
    """Against the largest value that the oracle's block and cross-attention store; within a factor of 200 of it."""
    m = synth.ModelShape(1, 256, 2, 128, 256, 64, 8, synth.BF16, 1, 1, (synth.ViewGroup(1, 1, 6, 7),), cond_len=20)
    blob = synth.make_weights(m)
    w = synth.split_block_weights(m, blob, 0)
    w["b_ada"] += 0.5
    w["bv"] -= 3.0
    orc = xo.XCacheOracle(m, synth.GateParams(), blob)
    cond = synth.condition_tokens(m)
    orc.set_condition(cond)
    a = np.full(8, action, np.float32)
    x = next(iter(synth.latent_stream(m, synth.StreamParams(1, 0.9, 0.02), 0, 1))).astype(np.float64)
    x[0] = 1e4 * np.eye(256)[3]  # a LayerNorm output of sqrt(C) in one column
    _, (_, v) = orc.block(0, x, orc.cond(500.0, a), None)

    def rows(weight, bias):
        return np.linalg.norm(weight.astype(np.float64), axis=1).max(), np.abs(bias).max()

    mod = rows(w["w_ada"][:2 * 256], w["b_ada"][:2 * 256])
    bound = rules.lib().self_bound(*mod, *rows(w["wv"], w["bv"]), 256, m.cond_dim, max(1.0, action))
    assert np.abs(v).max() <= bound <= 200 * np.abs(v).max()
    bound = rules.lib().cross_bound(*rows(w["wv_c"], w["bv_c"]), 256, float(np.abs(cond).max()))
    assert np.abs(orc.cross_kv[0][1]).max() <= bound <= 200 * np.abs(orc.cross_kv[0][1]).max()
    w["wv"][5, 7] = math.nan
    assert not rules.lib().bounded(16.6, rules.lib().self_bound(*mod, *rows(w["wv"], w["bv"]), 256, m.cond_dim, 1.0), 64)


def test_adaln_wave_rows():
    """8 rows per wave wherever 32 measured slower, 32 where 8 did (rows, 16-byte chunks per row)."""
    rows = rules.lib().wave_rows
    for n, chunks in ((12288, 18), (49152, 18), (49152, 33), (55296, 50), (73728, 32), (73728, 48), (147456, 40),
                      (147456, 56), (147456, 128), (368640, 64)):
        assert rows(n, chunks) == 8, (n, chunks)
    for n, chunks in ((73728, 9), (61440, 18), (122880, 18), (368640, 18), (147456, 24), (147456, 30), (73728, 33), (368640, 34),
                      (98304, 50)):
        assert rows(n, chunks) == 32, (n, chunks)


def test_gemm_f32_tiles():
    """The tile that measured fastest (M, N, K on 256 CUs), and both tiles' edges."""
    tile = rules.lib().f32_tile
    for want, cases in ((16, ((64, 384, 128), (64, 1024, 1024), (200, 512, 512), (512, 256, 1024), (700, 256, 256), (1100, 256, 64))),
                        (32, ((200, 768, 3072), (300, 768, 768), (512, 512, 512), (2048, 256, 256), (700, 3072, 1024),
                              (2048, 1536, 1536), (4096, 1024, 1024))),
                        (64, ((2048, 2304, 768), (4096, 1536, 512), (4096, 4608, 1536)))):
        for c in cases:
            assert tile(*c, 256) == want, c
    assert (tile(16, 8192, 512, 256), tile(16, 8193, 512, 256)) == (16, 32)
    assert (tile(16, 24576, 508, 256), tile(16, 24577, 508, 256)) == (16, 32)
    assert (tile(4096, 1024, 4, 256), tile(4096, 1025, 4, 256)) == (32, 64)


def test_f32_attention_waves():
    assert [rules.lib().f32_waves(k) for k in (1, 64, 65, 128, 129, 1 << 24)] == [1, 1, 2, 2, 4, 4]


def test_gemm_tiles_are_all_tested():
    """The tiles that the GPU test of the products names are the ones the rule picks, and every tile that an epilogue can
    take is among them."""
    import test_gpu_gemm_tiles as gt
    seen = {}
    for name, shape in gt.SHAPES.items():
        picked = {e: rules.tile(*p, 256) for e, p in gt.products(name).items()}
        assert tuple(picked.values()) == shape[4], name
        for e, t in picked.items():
            seen.setdefault(e, set()).add(t)
    everything = set(rules.TILES)
    assert seen == {"qkv": everything - {"64x64"}, "output": everything, "up": everything, "down": everything}


def test_products_without_a_kernel_are_refused():
    """(type, epilogue) pairs that no kernel serves: refused before anything is launched (no other kernel may read
    operands of the wrong type)."""
    from paper_2604_20289_amd import xcache as xcp
    launch = xcp.load_library()._ZN2xc11launch_gemmEiNS_7EpiModeEPKvS2_iiiRKNS_7EpiArgsEPKiP12ihipStream_t
    vp, i = ctypes.c_void_p, ctypes.c_int
    launch.restype, launch.argtypes = i, [i, i, vp, vp, i, i, i, ctypes.c_char_p, vp, vp]
    bias_f32, qkv = 0, 4
    f32, bf16 = 0, 1
    for dtype, mode in ((bf16, bias_f32), (f32, qkv)):
        assert launch(dtype, mode, None, None, 64, 128, 128, bytes(1024), None, None) == 1  # hipErrorInvalidValue
