"""Tile shapes of the bf16 projections against the CPU oracle: wide and small
tiles with ragged last row tiles, K of the fewest stages the rings handle
(128: two), of fewer stages than requests ahead and of many, in the QKV,
output, MLP-up and MLP-down epilogues.

Tolerance: relative L2 2e-2, the bf16 bar of the parity suite; the CPU side
computes in float32 with bf16 storage rounding."""
import numpy as np
import pytest

import rules
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# name: (hidden, heads, mlp, grid, the tiles the launcher picks on 256 CUs for QKV, output, MLP up and MLP down).  "deep":
# one workgroup per CU with a deep stage ring.  K = hidden, but mlp for MLP down
SHAPES = {
    "h384-L16000": (384, 3, 384, (1, 1, 125, 128), ("192x128", "128x128", "128x128", "128x128")),
    "h1152-L7020": (1152, 9, 1152, (2, 3, 26, 45), ("192x128", "128x128", "128x128", "128x128")),
    "h768-L16000": (768, 6, 768, (1, 1, 125, 128), ("192x128", "192x128", "192x128", "192x128")),
    "h2048-L6100": (2048, 16, 128, (1, 1, 61, 100), ("192x256", "192x256", "64x64", "192x128")),
    "h640-L5000": (640, 5, 1280, (2, 1, 50, 50), ("192x128", "64x128", "128x128", "128x128 deep")),
    "h1024-L1100": (1024, 8, 1024, (1, 1, 44, 25), ("64x128", "64x128", "64x128", "64x128")),
    "h256-L70": (256, 2, 1024, (1, 1, 7, 10), ("64x128", "64x128", "64x128", "64x64")),
    "h1024-L12479": (1024, 8, 128, (1, 1, 1, 12479), ("256x256", "256x256", "64x128", "256x256")),
    "h512-L16": (512, 4, 128, (1, 1, 4, 4), ("64x128", "64x64", "64x64", "64x128")),
    "h640-L6635": (640, 10, 640, (1, 1, 5, 1327), ("128x128", "192x128 deep", "192x128 deep", "192x128 deep")),
    "h768-L2927": (768, 6, 768, (1, 1, 1, 2927), ("128x128", "128x128 deep", "128x128 deep", "128x128 deep")),
    "h768-L10961": (768, 12, 1280, (1, 1, 97, 113), ("256x256", "192x128", "256x256", "192x256")),
    "h1920-L321": (1920, 15, 128, (1, 1, 3, 107), ("128x128 deep", "64x64", "64x64", "64x128")),
    "h1280-L1114": (1280, 10, 128, (1, 2, 1, 557), ("192x128 deep", "64x128", "64x64", "64x128")),
    "h1024-L4163": (1024, 16, 2048, (1, 1, 23, 181), ("256x256", "192x128 deep", "192x256", "192x128 deep")),
}


def products(name):
    """{epilogue: (M, N, K, columns of each of q, k, v)} of a shape's four products."""
    C, _, Dm, g, _ = SHAPES[name]
    L = g[0] * g[1] * g[2] * g[3]
    return {"qkv": (L, 3 * C, C, C), "output": (L, C, C, 0), "up": (L, Dm, C, 0), "down": (L, C, Dm, 0)}


@pytest.mark.parametrize("name", sorted(SHAPES))
def test_gemm_tiles(name):
    """One block, one pass: the output on sampled rows (all keys and values count)."""
    from lockstep import rel_l2
    from oracle import xcache_oracle as xo
    from paper_2604_20289_amd.xcache import XC_CACHE_KEYS, XC_CACHE_VALUES, XCache
    C, H, Dm, grid, tiles = SHAPES[name]
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert [rules.tile(*p, cus) for p in products(name).values()] == list(tiles)
    m = synth.ModelShape(1, C, H, C // H, Dm, 256, 16, synth.BF16, 1, 1, (synth.ViewGroup(*grid),))
    gate = synth.GateParams(front_anchors=0)
    blob = synth.make_weights(m)
    w = synth.split_block_weights(m, blob, 0)
    w["b_ada"] += 0.5
    L = m.tokens
    x = next(iter(synth.latent_stream(m, synth.StreamParams(1, 0.9, 0.02), 0, 1)))
    a = next(iter(synth.action_stream(m, synth.StreamParams(1, 0.9, 0.02), 0, 1)))
    rows = np.unique(np.clip(np.r_[np.arange(0, L, 997), [1, 31, 32, 191, 192, 255, 256, L - 193, L - 33, L - 2, L - 1]], 0, L - 1))
    xc = XCache(m, gate, blob, torch.cuda.current_stream().cuda_stream)
    try:
        xd = torch.from_numpy(x).cuda()
        yd = torch.empty_like(xd)
        xc.forward_chunk(0, 1000.0, a, xd, yd)
        k = torch.empty(L * C, dtype=torch.float32, device="cuda")
        v = torch.empty_like(k)
        xc.read_cache(XC_CACHE_KEYS, 0, 0, k)
        xc.read_cache(XC_CACHE_VALUES, 0, 0, v)
        got = yd.cpu().numpy()
        k, v = (t.cpu().numpy().reshape(H, L, C // H) for t in (k, v))
    finally:
        xc.close()
    orc = xo.XCacheOracle(m, gate, blob, np.float32)
    c = orc.cond(1000.0, a)
    want, (ko, vo) = orc.block(0, x.astype(np.float32), c, rows)
    errs = {"y-x": rel_l2(got[rows] - x[rows], want - x[rows]), "K": rel_l2(k, ko), "V": rel_l2(v, vo)}
    print(f"[gemm tiles] {name} L={L}: " + " ".join(f"{n} {e:.2e}" for n, e in errs.items()), flush=True)
    for n, e in errs.items():
        assert e <= 2e-2, (n, e)
