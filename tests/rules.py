"""The host-side dispatch rules (csrc/xc_rules.h), compiled with the host
compiler and called through ctypes."""
import ctypes
import functools
import os
import subprocess
import tempfile

import numpy as np

from paper_2604_20289_amd import build

SHIM = r"""
#include "xc_rules.h"
using namespace xc;
extern "C" {
float score_bound(const float* gq, const float* gk, int D, int rope) { return qk_score_bound(gq, gk, D, rope != 0); }
double self_bound(double mod_norm, double mod_bias, double v_norm, double v_bias, int C, int Dc, double cond_max) {
  return self_value_bound({mod_norm, mod_bias}, {v_norm, v_bias}, C, Dc, cond_max);
}
double cross_bound(double v_norm, double v_bias, int C, double cond_max) {
  return cross_value_bound({v_norm, v_bias}, C, cond_max);
}
int wave_rows(long long rows, int chunks) { return adaln_wave_rows(rows, chunks); }
int f32_waves(long long Lk) { return attention_f32_waves(Lk); }
int wide_waves(int L, long long Lk, int D, long long items, int cus) { return attention_wide_waves(L, Lk, D, items, cus); }
int splits(long long items, long long tiles, long long slots, long long most) {
  return attention_split_count(items, tiles, slots, most);
}
int f32_tile(int M, int N, int K, int cus) { return gemm_f32_tile(M, N, K, cus); }
int tile(int M, int N, int K, int C, int cus) { return pick_tile(M, N, K, C, cus); }
int bounded(float score, double value, long long Lk) { return attention_bounded(score, value, Lk); }
}
"""


@functools.lru_cache(None)
def lib():
    d = tempfile.mkdtemp(prefix="xc_rules_")
    src, so = os.path.join(d, "shim.cpp"), os.path.join(d, "shim.so")
    with open(src, "w") as f:
        f.write(SHIM)
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-shared", "-fPIC", "-I", build.CSRC, src, "-o", so],
                   check=True)
    out = ctypes.CDLL(so)
    f, d, i, ll = ctypes.c_float, ctypes.c_double, ctypes.c_int, ctypes.c_longlong
    p = np.ctypeslib.ndpointer(np.float32, flags="C_CONTIGUOUS")
    for name, res, args in (("score_bound", f, [p, p, i, i]), ("self_bound", d, [d, d, d, d, i, i, d]),
                            ("cross_bound", d, [d, d, i, d]), ("bounded", i, [f, d, ll]), ("wave_rows", i, [ll, i]),
                            ("f32_waves", i, [ll]), ("tile", i, [i, i, i, i, i]), ("splits", i, [ll, ll, ll, ll]),
                            ("f32_tile", i, [i, i, i, i]), ("wide_waves", i, [i, ll, i, ll, i])):
        getattr(out, name).restype, getattr(out, name).argtypes = res, args
    return out


TILES = ["64x64", "64x128", "128x128 deep", "128x128", "192x128 deep", "192x128", "256x256", "192x256"]


def tile(M, N, K, C, cus):
    """The tile of a bf16 product (C: columns of each of q, k, v in the QKV product, else 0)."""
    return TILES[lib().tile(M, N, K, C, cus)]
