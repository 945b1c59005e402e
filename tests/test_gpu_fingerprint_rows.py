"""The gate's comparison with many fingerprint rows: several row chunks per
camera, chunks that span cameras and view groups, every token sampled; both
dtypes, decisions and reported metrics against the CPU oracle."""
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("budget", [31, 33, 150, 1000])
@pytest.mark.parametrize("dtype", [synth.F32, synth.BF16])
def test_fingerprint_budgets(dtype, budget):
    from lockstep import Lockstep
    m = synth.ModelShape(2, 256, 4, 64, 256, 64, 8, dtype, 2, 2,
                         (synth.ViewGroup(2, 3, 7, 9), synth.ViewGroup(1, 2, 5, 11)))
    w = synth.Workload("fingerprint-rows", m, synth.GateParams(front_anchors=0, fp_budget=budget, adaptive=0,
                                                               tau_cos_fixed=0.9, tau_dev=10.0),
                       synth.StreamParams(4, 0.999, 0.02))
    ls = Lockstep(w)
    try:
        st = ls.run(4, **({"tol_abs": 1e-4} if dtype == synth.F32 else {"tol_rel_l2": 2e-2}))
        assert st["skips"] > 0
        print(f"[rows] {dtype} budget {budget}: skips {st['skips']} worst {max(ls.worst.values()):.2e}", flush=True)
    finally:
        ls.close()


@pytest.mark.parametrize("groups", [5, 8])
def test_many_groups(groups):
    """More records than the decision reads in one round (some 5000 and 9000), group counts that do and do not divide its
    threads."""
    from lockstep import Lockstep
    m = synth.ModelShape(2, 1024, 8, 128, 128, 64, 8, synth.BF16, 2, 1,
                         tuple(synth.ViewGroup(1, 1, 9 + i % 3, 11) for i in range(groups)))
    w = synth.Workload(f"fingerprint-{groups}-groups", m,
                       synth.GateParams(front_anchors=0, fp_budget=1000, adaptive=0, tau_cos_fixed=0.9, tau_dev=10.0),
                       synth.StreamParams(3, 0.999, 0.02))
    ls = Lockstep(w)
    try:
        st = ls.run(3, tol_rel_l2=2e-2)
        assert st["skips"] > 0
        print(f"[rows] {groups} groups: skips {st['skips']} worst {max(ls.worst.values()):.2e}", flush=True)
    finally:
        ls.close()
