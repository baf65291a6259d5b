"""The rule that picks 128- or 256-row workgroups for a launch of the attention kernel, asked on the CPU: a row's bits do not
depend on the shape, so no result shows which one ran."""
import ctypes
import os
import subprocess

import pytest

import paper_2410_02367_amd as sage
from paper_2410_02367_amd import build

SHIM = """#include "sage_shape.h"
extern "C" int small_workgroups(int D, int BH, int Nq, int N, int causal, int n_splits, int chunk) {
    return sage::small_workgroups(D, BH, Nq, N, causal != 0, n_splits, chunk);
}
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    """rows of a workgroup: f(D, slabs, Nq, N, causal, n_splits, chunk)"""
    at = tmp_path_factory.mktemp("shape")
    src, lib = at / "shape.cpp", at / "shape.so"
    src.write_text(SHIM)
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I" + build.CSRC, "-o", str(lib), str(src)], check=True)
    f = ctypes.CDLL(str(lib)).small_workgroups
    return lambda *a: 128 if f(*(int(x) for x in a)) else 256


# (slabs, Nq, Nkv, requested chunks, rows): the cases that test_gpu_split.py runs, and two of those that the rule was measured at
CHUNKS = [(13, 130, 40000, 0, 256), (20, 250, 30000, 0, 256), (65, 129, 5200, 2, 256), (40, 300, 16500, 0, 128), (12, 500, 10000, 4, 128),
          (32, 512, 16384, 0, 256), (40, 640, 12000, 0, 128)]


@pytest.mark.parametrize("slabs,Nq,Nkv,req,rows", CHUNKS)
def test_chunks_under_a_mask(rule, slabs, Nq, Nkv, req, rows):
    from test_gpu_split import SHAPES_OF_CHUNKS, chunk_starts
    assert (slabs, Nq, Nkv) in [s[:3] for s in SHAPES_OF_CHUNKS] or Nq in (512, 640)
    n = sage.sage_attn_split_count(1, slabs, Nq, Nkv, True, req)
    chunk = chunk_starts(1, slabs, Nq, Nkv, True, req or n)[1]
    assert n > 1 and chunk > 2048
    assert rule(128, slabs, Nq, Nkv, True, n, chunk) == rows


# (D, slabs, Nq, N, causal, rows): either side of every line of the rule
WHOLE = [(64, 500, 9000, 9000, False, 128), (64, 500, 9000, 9000, True, 128),
         (128, 128, 4096, 2048, False, 128), (128, 86, 4096, 4096, False, 128), (128, 12, 3000, 3000, False, 256),
         (128, 12, 6000, 6000, False, 128), (128, 30, 3000, 3000, False, 128), (128, 46, 3800, 3800, False, 256),
         (128, 96, 640, 2816, False, 128), (128, 128, 4096, 4096, False, 256),
         (128, 128, 4096, 4096, True, 128), (128, 16, 5000, 5000, True, 128), (128, 32, 16384, 16384, True, 256),
         (128, 31, 4097, 4097, True, 256), (128, 30, 4097, 4097, True, 128)]


@pytest.mark.parametrize("D,slabs,Nq,N,causal,rows", WHOLE)
def test_whole_sequences(rule, D, slabs, Nq, N, causal, rows):
    assert rule(D, slabs, Nq, N, causal, 1, 0) == rows
