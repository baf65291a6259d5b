"""Launches of at most one 128-row workgroup per compute unit at D = 64: two sets of wavefronts share a workgroup's rows, each
with half of the keys.  Against the CPU oracle where the halves can go wrong, and the rule that picks them on the CPU."""
import ctypes
import subprocess

import numpy as np
import pytest
import torch

import oracle
import paper_2410_02367_amd as sage
import sage_inputs as si
from gpu_util import assert_output_close, to_dev
from paper_2410_02367_amd import build

SHIM = """#include "sage_shape.h"
extern "C" int two_halves(int D, int BH, int Nq, int N, int n_splits) {
    return sage::two_halves(D, BH, Nq, N, n_splits);
}
"""


@pytest.mark.parametrize("D,slabs,Nq,N,n_splits,two", [
    (64, 1, 1024, 1024, 1, True), (64, 1, 1023, 1023, 1, False), (64, 32, 1024, 1024, 1, True), (64, 32, 1025, 1025, 1, False),
    (64, 256, 128, 1500, 1, True), (64, 257, 128, 1500, 1, False), (64, 1, 300, 9000, 2, False), (128, 1, 4096, 4096, 1, False)])
def test_the_rule_for_two_sets(tmp_path, D, slabs, Nq, N, n_splits, two):
    src, lib = tmp_path / "shape.cpp", tmp_path / "shape.so"
    src.write_text(SHIM)
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I" + build.CSRC, "-o", str(lib), str(src)], check=True)
    assert bool(ctypes.CDLL(str(lib)).two_halves(D, slabs, Nq, N, n_splits)) == two


# (slabs, Nq, Nkv, causal, block_q, block_k, rising).  1024, 1025, 1087: sets of the same number of keys, a second set that ends
# on a tile of one key or one that lacks one; 64-key blocks and 128-key ones, whose boundary the cut keeps to; causal: rows whose
# first keys are the first set's alone (both sets then walk all keys), queries that are the last of the keys; rising: a maximum
# that rises in either half.
CASES = [
    (2, 1024, 1024, False, 128, 64, False), (2, 1025, 1025, False, 64, 128, False), (1, 1087, 1087, False, 1, 1, False),
    (3, 1153, 1153, False, 128, 128, False), (2, 1500, 1500, False, 128, 64, True), (2, 1024, 1024, True, 128, 64, False),
    (2, 1089, 1089, True, 128, 128, False), (1, 1111, 1111, True, 1, 1, False), (2, 1200, 1200, True, 64, 64, True),
    (2, 130, 1400, True, 128, 64, False), (2, 90, 1025, True, 32, 128, True), (3, 333, 1050, False, 128, 1, False),
]


@pytest.mark.gpu
@pytest.mark.parametrize("slabs,Nq,Nkv,causal,bq,bk,rising", CASES)
def test_two_sets_match_the_oracle(slabs, Nq, Nkv, causal, bq, bk, rising):
    print(f"[case] {slabs} x {Nq} against {Nkv} causal={causal} scales {bq}x{bk} rising={rising}", flush=True)
    w = si.custom("halves", 1, slabs, max(Nq, Nkv), 64, causal, bq, bk, k_noise=1.0, k_bias=3.0, seed=si.BASE_SEED + 1400 + Nkv)
    q, k, v = si.full(w)
    q, k, v = (np.ascontiguousarray(x[:, :, :n]) for x, n in ((q, Nq), (k, Nkv), (v, Nkv)))
    if rising:
        k = (k.astype(np.float32) * np.linspace(0.5, 8.0, Nkv, dtype=np.float32)[None, None, :, None]).astype(np.float16)
    k_i8, k_scale, _ = sage.sage_smooth_quant_k(to_dev(k), bk)
    q_i8, q_scale = sage.sage_quant_q(to_dev(q), w.sm_scale, bq)
    o = sage.sage_attn_cross_fwd(q_i8, q_scale, k_i8, k_scale, to_dev(v), causal, w.sm_scale, bq, bk)
    torch.cuda.synchronize()
    kq, ks, _ = oracle.smooth_quant_k(k, bk)
    qq, qs = oracle.quant_q(q, w.sm_scale, bq)
    lq, lk = 128 if bq == 1 else max(bq, 64), 64 if bk == 1 else max(bk, 64)
    ref = oracle.attn_l2_cross(qq, qs, kq, ks, v, causal, lq, lk, gran_q=bq, gran_k=bk)
    assert_output_close(o.cpu().numpy(), ref, f"{Nq} x {Nkv}")
