"""The wait states around the inline-assembly MFMAs of the bounded attention
kernel, read from its assembly: as built, and under two instruction
schedulers that move register arithmetic much further than the default one
does (a wait that names no registers does not hold there)."""
import os
import subprocess

import pytest

from mfma_hazards import functions, violations
from paper_2604_20289_amd import build

SCHEDULERS = {"default": [], "ilpmax": ["-mllvm", "-misched=ilpmax"],
              "iterative-ilp": ["-mllvm", "-misched=gcn-iterative-ilp"]}


@pytest.mark.parametrize("scheduler", sorted(SCHEDULERS))
def test_bounded_attention(scheduler, tmp_path):
    out = str(tmp_path / "attention.s")
    r = subprocess.run([build._hipcc(), *build.COMMON_FLAGS, *SCHEDULERS[scheduler], "-x", "hip", "-S", "--cuda-device-only",
                        os.path.join(build.CSRC, "xc_attention.hip"), "-o", out], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    kernels = functions(open(out).read(), "attn_bounded_kernel")
    assert len(kernels) == 2  # head dims 64 and 128
    for name, body in kernels.items():
        assert sum(t.startswith("v_mfma") for _, t in body) >= 100
        assert violations(body) == [], name


MFMA = "v_mfma_f32_32x32x16_bf16 v[0:15], v[20:23], v[24:27], v[0:15]"


@pytest.mark.parametrize("body,early", [
    ([MFMA, "s_nop 15", "v_exp_f32_e32 v30, v3"], 1),                                      # read 16 wait states later
    ([MFMA, "s_nop 15", "s_nop 7", "v_exp_f32_e32 v30, v3"], 0),
    ([MFMA, "s_nop 15", "v_mov_b32_e32 v3, v30"], 1),                                      # overwritten
    ([MFMA, MFMA], 0),                                                                     # accumulates
    ([MFMA, "v_mfma_f32_32x32x16_bf16 v[8:23], v[32:35], v[24:27], v[8:23]"], 1),          # overlaps
    (["v_cvt_pk_bf16_f32 v25, v30, v31", MFMA], 1),                                        # operand just written
    (["v_cvt_pk_bf16_f32 v25, v30, v31", "s_nop 1", MFMA], 0),
    # around a loop: the read at its top follows the MFMA at its bottom
    ([".LBB0_1:", "v_exp_f32_e32 v30, v3", "s_nop 15", "s_nop 15", MFMA, "s_cbranch_scc1 .LBB0_1", "s_endpgm"], 1),
    (["s_cbranch_scc1 .LBB0_1", MFMA, ".LBB0_1:", "v_exp_f32_e32 v30, v3", "s_endpgm"], 1),  # on one of two ways
])
def test_the_reader(body, early):
    assert len(violations(list(enumerate(body)))) == early
