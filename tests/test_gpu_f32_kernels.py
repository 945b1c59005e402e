"""The float32 kernels where their dispatch changes, against the CPU oracle
(max-abs 1e-4, the bar of the float32 model): products on 16- and 32-square
tiles and on the staged 64 x 64 ones, K that is no multiple of 16 or of 4,
ragged rows and columns; attention with 16-byte and scalar rows, fewer keys
than a chunk, fewer chunks than waves and several per wave."""
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# name: (hidden, heads, mlp, kv_window, grid).  Tiles of 16 x 16 on 256 CUs: up to 1536 (512 with K of 512 and more) take
# 16-square tiles, up to 16384 32-square ones (h256-L300: output 304, QKV 912, MLP up 1216, MLP down 304;
# h512-L1100: output 2208, QKV 6624, MLP up 8832; h512-L2050: QKV 12384, MLP up 17028 on 64 x 64)
MODELS = {
    "h128-L64": (128, 4, 512, 2, (1, 4, 4, 4)),
    "h256-L300": (256, 4, 1024, 2, (2, 3, 5, 10)),
    "h512-L1100": (512, 8, 2048, 1, (1, 1, 25, 44)),
    "h512-L2050": (512, 8, 2112, 1, (1, 1, 41, 50)),
    "h84-d28-mlp52": (84, 3, 52, 3, (1, 1, 7, 11)),       # K = 84 and 52: part of a 16-deep chunk
    "h12-d6-mlp30": (12, 2, 30, 2, (1, 1, 3, 11)),        # rows of no multiple of 16 bytes (MLP down, heads)
    "h128-d128-L20": (128, 1, 130, 4, (1, 1, 4, 5)),      # one head of 128, 20 to 80 keys
}


@pytest.mark.parametrize("rope", [0, 1])
@pytest.mark.parametrize("name", sorted(MODELS))
def test_f32_kernels(name, rope):
    from lockstep import Lockstep
    C, H, Dm, window, grid = MODELS[name]
    m = synth.ModelShape(2, C, H, C // H, Dm, 64, 8, synth.F32, 1, window, (synth.ViewGroup(*grid),), rope=rope,
                         cond_len=9 if rope else 0)
    w = synth.Workload(f"f32-{name}", m, synth.GateParams(), synth.StreamParams(window + 1, 0.97, 0.02))
    ls = Lockstep(w)
    try:
        ls.run(w.stream.n_chunks, tol_abs=1e-4)
        print(f"[f32] {name} rope={rope}: worst {max(ls.worst.values()):.2e}", flush=True)
    finally:
        ls.close()


@pytest.mark.parametrize("blocks", [39, 40])
def test_adaln_rows_per_wave(blocks):
    """60840 modulation rows (8 per wave) and 62400 (32 per wave), neither a whole number of workgroups."""
    from lockstep import Lockstep
    m = synth.ModelShape(blocks, 260, 5, 52, 64, 64, 8, synth.F32, 1, 1, (synth.ViewGroup(1, 1, 3, 3),))
    w = synth.Workload(f"f32-adaln-{blocks}", m, synth.GateParams(), synth.StreamParams(1, 0.97, 0.02))
    ls = Lockstep(w)
    try:
        ls.run(1, tol_abs=1e-4)
        print(f"[f32] adaLN {6 * 260 * blocks} rows: worst {max(ls.worst.values()):.2e}", flush=True)
    finally:
        ls.close()


# one, two and four waves per query at the edges of their chunks, scalar and 16-byte rows; one wave's rows of 1, 5 and 17
# sixteen-byte chunks (it loads four at a time) and 1 to 3 keys past a multiple of four
WAVES = ([(d, c) for d in (6, 64, 128) for c in (1, 63, 64, 65, 128, 129, 257)]
         + [(d, c) for d in (4, 20, 68) for c in (2, 3, 4, 61, 62)])


@pytest.mark.parametrize("head_dim,cond", WAVES)
def test_attention_waves(head_dim, cond):
    """Cross-attention to few keys."""
    from lockstep import Lockstep
    m = synth.ModelShape(1, 2 * head_dim, 2, head_dim, 64, 64, 8, synth.F32, 1, 1, (synth.ViewGroup(1, 1, 3, 7),),
                         cond_len=cond)
    w = synth.Workload(f"f32-waves-d{head_dim}-c{cond}", m, synth.GateParams(), synth.StreamParams(1, 0.97, 0.02))
    blob = synth.make_weights(m)
    t = synth.split_block_weights(m, blob, 0)
    t["wv_c"] *= 8
    t["wo_c"] *= 8
    ls = Lockstep(w, weights=blob)
    try:
        ls.run(1, tol_abs=1e-4)
        print(f"[f32] d={head_dim} {cond} keys: worst {max(ls.worst.values()):.2e}", flush=True)
    finally:
        ls.close()
