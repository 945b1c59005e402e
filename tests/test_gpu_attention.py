"""The two attention kernels (scores bounded by the RMSNorm gains, and the
running-maximum one) against the CPU oracle where they can go wrong: one key
tile, every phase of the three-slot tile ring, ragged last tiles and query
blocks, both head dims, cross-attention's own gains.

Tolerance: relative L2 2e-2 on y, y - x and the caches, the bf16 bar of the
parity suite.  The projections are scaled so that attention carries most of
y - x."""
import math

import numpy as np
import pytest

import rules
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# tokens: with a window of 3 chunks the passes see 1 / 2 / 2, 2 / 4 / 5, 3 / 5 / 8
# and 5 / 9 / 13 key tiles of 64
TOKENS = {40: (1, 1, 2, 20), 100: (1, 2, 5, 10), 150: (1, 3, 5, 10), 257: (1, 1, 1, 257), 300: (2, 3, 5, 10)}
# gains 1: |score| <= sqrt(128) log2(e) = 16.3; gains 2.5: 6.25 times that, past the bound of 64 (up to 128 queries the
# running maximum serves both)
GAINS = {"bounded": 1.0, "running-max": 2.5}


def _workload(tokens, head_dim, **kw):
    return synth.Workload(
        f"attention-h256-d{head_dim}-L{tokens}",
        synth.ModelShape(1, 256, 256 // head_dim, head_dim, 256, 256, 16, synth.BF16, 1, 3,
                         (synth.ViewGroup(*TOKENS[tokens]),), **kw),
        synth.GateParams(), synth.StreamParams(3, 0.97, 0.02))


def _weights(m, gain, cross_gain=1.0):
    blob = synth.make_weights(m)
    for b in range(m.n_blocks):
        w = synth.split_block_weights(m, blob, b)
        w["wv"] *= 4
        w["wo"] *= 8
        w["gq"][:] = gain
        w["gk"][:] = -gain  # the bound takes magnitudes
        if m.cond_len:
            w["wv_c"] *= 4
            w["wo_c"] *= 4
            w["gq_c"][:] = cross_gain
            w["gk_c"][:] = cross_gain
    return blob


def _run(w, blob, **kw):
    from lockstep import Lockstep
    ls = Lockstep(w, weights=blob, compute=np.float64)
    try:
        ls.run(w.stream.n_chunks, tol_rel_l2=2e-2, **kw)
        print(f"[attention] {w.name}: worst {max(ls.worst.values()):.2e}", flush=True)
    finally:
        ls.close()


@pytest.mark.parametrize("tokens", sorted(TOKENS))
@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("kernel", sorted(GAINS))
def test_attention_kernels(kernel, head_dim, tokens):
    w = _workload(tokens, head_dim)
    _run(w, _weights(w.model, GAINS[kernel]))


@pytest.mark.parametrize("gain,cross_gain", [(1.0, 2.5), (2.5, 1.0)])
def test_attention_kernels_rope_and_cross(gain, cross_gain):
    """Each attention of a block takes the kernel that its own gains allow; 70 condition tokens leave a ragged tile."""
    w = _workload(150, 128, rope=1, cond_len=70)
    _run(w, _weights(w.model, gain, cross_gain))


def test_uneven_gains_with_rotation():
    """A rotation mixes the two dimensions of a pair: gains that alternate between 4 and 1/4 (products of 1 in every
    dimension, pair bound 16) must not be taken as bounded by 1."""
    w = _workload(150, 128, rope=1)
    blob = _weights(w.model, 1.0)
    t = synth.split_block_weights(w.model, blob, 0)
    t["gq"][0::2], t["gq"][1::2] = 4.0, 0.25
    t["gk"][0::2], t["gk"][1::2] = 0.25, 4.0
    _run(w, blob)


@pytest.mark.parametrize("cond", [5, 64])
@pytest.mark.parametrize("head_dim", [64, 128])
def test_one_key_tile(head_dim, cond):
    """Cross-attention without a running maximum over a single key tile, ragged and whole."""
    w = _workload(150, head_dim, cond_len=cond)
    _run(w, _weights(w.model, 1.0))


@pytest.mark.parametrize("cond", [100, 128])
def test_two_key_tiles_many_items(cond):
    """Two key tiles, 17 query tiles in 16 heads of 64: more items than CUs, so no running maximum."""
    m = synth.ModelShape(1, 1024, 16, 64, 128, 64, 8, synth.BF16, 1, 1, (synth.ViewGroup(1, 1, 1, 4100),), cond_len=cond)
    w = synth.Workload(f"attention-h1024-d64-c{cond}", m, synth.GateParams(), synth.StreamParams(1, 0.97, 0.02))
    assert rules.lib().wide_waves(4100, cond, 64, 16 * 17, torch.cuda.get_device_properties(0).multi_processor_count)
    blob = _weights(m, 1.0)
    from lockstep import Lockstep
    ls = Lockstep(w, weights=blob, compute=np.float32)
    try:
        ls.run(1, tol_rel_l2=2e-2)
        print(f"[attention] {w.name}: worst {max(ls.worst.values()):.2e}", flush=True)
    finally:
        ls.close()


def _lean(w, sign, suffix=""):
    """Biases that turn every query (and, times sign, every key) towards one direction, so all scores lie near the
    bound of their gains times sign."""
    s = np.where(np.arange(w["bq"].size) % 3 == 0, -1.0, 1.0)
    w["bq" + suffix][:] = s
    w["bk" + suffix][:] = sign * s


class _Scores:
    """Records the range of the oracle's scores in log2 units, and the lowest maximum of a row."""

    def __init__(self, monkeypatch):
        from oracle import xcache_oracle as xo
        self.lo, self.hi, self.row_max = math.inf, -math.inf, math.inf
        attend = xo.softmax_attention

        def record(q, k, v):
            s = (q @ k.T) * (math.log2(math.e) / math.sqrt(q.shape[1]))
            self.lo, self.hi = min(self.lo, s.min()), max(self.hi, s.max())
            self.row_max = min(self.row_max, s.max(axis=1).min())
            return attend(q, k, v)

        monkeypatch.setattr(xo, "softmax_attention", record)


def _lean_workload(head_dim, cross, gain, sign):
    """One direction for every query and key of the self- or the cross-attention, with these gains."""
    w = _workload(150, head_dim, cond_len=70 if cross else 0)
    blob = _weights(w.model, 1.0 if cross else gain, gain)
    s = "_c" if cross else ""
    t = synth.split_block_weights(w.model, blob, 0)
    _lean(t, sign if cross else -sign, s)  # (the gains of k have the other sign)
    bound = rules.lib().score_bound(np.ascontiguousarray(t["gq" + s]), np.ascontiguousarray(t["gk" + s]), head_dim, 0)
    return w, blob, t, s, bound


@pytest.mark.parametrize("cross", [False, True])
@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("sign", [1, -1])
def test_scores_at_the_bound(sign, head_dim, cross, monkeypatch):
    """The largest gains that the kernel without a maximum takes (bound just under 64), all scores near it or near minus
    it: probabilities of 2^50 to 2^64, or their reciprocals."""
    w, blob, _, _, bound = _lean_workload(head_dim, cross, 1.955 if head_dim == 128 else 2.325, sign)
    assert 63 < bound <= 64
    sc = _Scores(monkeypatch)
    _run(w, blob)
    assert 50 < (sc.hi if sign > 0 else -sc.lo) < 64


@pytest.mark.parametrize("cross", [False, True])
@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("sign", [1, -1])
def test_scores_past_the_range(sign, head_dim, cross, monkeypatch):
    """Probabilities of 2^140 and more, or of less than 2^-150 for every key: an unsubtracted 2^s is infinite, or their sum 0."""
    w, blob, _, _, bound = _lean_workload(head_dim, cross, 3.4 if head_dim == 128 else 4.1, sign)
    assert bound > 64
    sc = _Scores(monkeypatch)
    _run(w, blob)
    assert sc.hi > 140 if sign > 0 else sc.row_max < -150


def test_rotated_scores_past_the_range(monkeypatch):
    """Gains of 3.4 in the even and 1 / 3.4 in the odd dimensions of q, the reverse in k: products of 1 in every dimension (a
    bound of 16.6), but queries along the even and keys along the odd dimensions meet under a rotation, at 2^140 and more."""
    w = _workload(150, 128, rope=1, rope_theta=1.01)  # every pair turns by about the same angle
    blob = _weights(w.model, 1.0)
    t = synth.split_block_weights(w.model, blob, 0)
    for name, even in (("q", 3.4), ("k", 1 / 3.4)):
        t["g" + name][0::2], t["g" + name][1::2] = even, 1 / even
        t["b" + name][0::2], t["b" + name][1::2] = (4.0, 0.0) if name == "q" else (0.0, 4.0)
    sc = _Scores(monkeypatch)
    _run(w, blob)
    assert sc.hi > 140


@pytest.mark.parametrize("cross", [False, True])
@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("sign", [1, -1])
def test_value_range(sign, head_dim, cross, monkeypatch):
    """All scores near 50 with values of 2^105, or near -50 with values of 2^-105: the products leave the range of a float
    unless the row's maximum is subtracted, which the bound on the values decides."""
    w, blob, t, s, _ = _lean_workload(head_dim, cross, 1.9 if head_dim == 128 else 2.25, sign)
    for name, scale in (("wv", 2.0 ** (105 * sign)), ("bv", 2.0 ** (105 * sign)), ("wo", 2.0 ** (-105 * sign))):
        t[name + s] *= scale
    sc = _Scores(monkeypatch)
    _run(w, blob)
    assert 40 < (sc.hi if sign > 0 else -sc.lo) < 64


@pytest.mark.parametrize("row", [0, 255])
def test_value_range_of_one_row(row):
    """Values of 2^105 in one column only, the first and the last."""
    w, blob, t, _, _ = _lean_workload(128, False, 1.9, 1)
    t["wv"][row] *= 2.0 ** 105
    t["bv"][row] *= 2.0 ** 105
    t["wo"][:, row] *= 2.0 ** -105
    _run(w, blob)
