"""Scores that leave the range of the running maximum: it is kept until a tile's exceeds it by more than 2^8.  Keys that grow
along the sequence (every block with another scale, so that the grid of the maximum changes too), one far larger key in the
middle or at the end, or scores so wide that a row rests on one key, in every shape of the attention kernel, against the
oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2410_02367_amd as sage
import sage_inputs as si
from gpu_util import assert_output_close, to_dev

pytestmark = pytest.mark.gpu

# B, H, Nq, Nkv, D, causal, block_q, block_k
SHAPES = [
    (1, 2, 513, 513, 64, False, 128, 64), (1, 2, 700, 700, 64, True, 1, 64), (1, 2, 1105, 1105, 64, True, 32, 128), (1, 2, 600, 600, 64, True, 1, 1),
    (1, 2, 300, 300, 128, False, 64, 64), (1, 2, 577, 577, 128, True, 128, 128), (1, 2, 640, 640, 128, False, 1, 1),
    (1, 2, 33, 1500, 128, True, 128, 64), (1, 3, 200, 3000, 64, False, 128, 64),       # keys in chunks
    (5, 13, 513, 513, 64, False, 128, 64), (5, 13, 577, 577, 64, True, 128, 128), (5, 13, 520, 520, 64, True, 1, 1),  # D = 64, one set of wavefronts
    (1, 17, 2100, 2100, 128, False, 128, 64), (2, 29, 2300, 4200, 128, True, 128, 64),  # workgroups of 256 rows
]


def keys(kind, k, q):
    N = k.shape[2]
    if kind == "growing":
        return k * np.geomspace(0.1, 10.0, N)[:, None]
    if kind == "wide":
        return k * 30.0
    at = {"middle": N // 2, "last": N - 1, "second tile": 64}[kind]
    k = k.copy()
    # the side on which the last query's score is large
    k[:, :, at] *= 14.0 * np.sign((k[:, :, at] * q[:, :, -1]).sum(-1, keepdims=True))
    return k


def raised_rows(qq, qs, kq, ks, causal, bq, bk):
    """Rows of a slab with a tile whose scores exceed all of the tiles before it by more than 8 in the exponent of 2."""
    Nq, N = len(qq), len(kq)
    s = (qq.astype(np.float64) @ kq.astype(np.float64).T) * np.repeat(qs, bq)[:Nq, None] * np.repeat(ks, bk)[None, :N] * np.log2(np.e)
    if causal:
        s[np.arange(N)[None, :] > np.arange(Nq)[:, None] + N - Nq] = -np.inf
    tiles = np.pad(s, ((0, 0), (0, -N % 64)), constant_values=-np.inf).reshape(Nq, -1, 64).max(2)
    return int((tiles[:, 1:] > np.maximum.accumulate(tiles, 1)[:, :-1] + 8).any(1).sum())


@pytest.mark.parametrize("kind", ["growing", "middle", "last", "second tile", "wide"])
@pytest.mark.parametrize("B, H, Nq, Nkv, D, causal, bq, bk", SHAPES)
def test_scores_far_above_those_of_the_first_tile(kind, B, H, Nq, Nkv, D, causal, bq, bk):
    if H > 13 and kind != "growing":
        pytest.skip("the large shapes run once")
    print(f"[case] {kind} B{B} H{H} Nq{Nq} Nkv{Nkv} D{D} causal={causal} scales {bq}x{bk}", flush=True)
    rng = np.random.default_rng(si.BASE_SEED + Nkv + D)
    q = (3.0 * rng.standard_normal((B, H, Nq, D))).astype(np.float16)
    k = keys(kind, rng.standard_normal((B, H, Nkv, D)), q.astype(np.float64)).astype(np.float16)
    # rows are all but a single value here: below 2, where one unit of the fp16 result is half of the tolerance
    v = np.clip(rng.standard_normal((B, H, Nkv, D)), -1.99, 1.99).astype(np.float16)
    sm = D ** -0.5
    out = sage.sageattn(to_dev(q), to_dev(k), to_dev(v), causal, sm, bq, bk).cpu().numpy()
    kq, ks, _ = oracle.smooth_quant_k(k, bk)
    qq, qs = oracle.quant_q(q, sm, bq)
    lq, lk = max(bq, 64) if bq != 1 else 128, max(bk, 64) if bk != 1 else 64
    heads = [(0, 0), (B - 1, H - 1)]
    assert sum(raised_rows(qq[b, h], qs[b, h], kq[b, h], ks[b, h], causal, bq, bk) for b, h in heads) > 0
    for b, h in heads:
        one = lambda x: np.ascontiguousarray(x[b:b + 1, h:h + 1])
        ref = oracle.attn_l2_cross(one(qq), one(qs), one(kq), one(ks), one(v), causal, lq, lk, gran_q=bq, gran_k=bk)
        assert_output_close(one(out), ref, f"{kind}, head {b} {h}")


@pytest.mark.parametrize("factor", [1e-9, 1e-4, 1e-2, 1.0])
@pytest.mark.parametrize("causal", [False, True])
def test_small_scores(factor, causal):
    """However small the scores, and with them the constant that their factor is folded with, the result is the oracle's."""
    print(f"[case] key scales x {factor}, causal={causal}", flush=True)
    w = si.custom("small", 1, 2, 1500, 128, causal, seed=si.BASE_SEED + 1500)
    q, k, v = si.full(w)
    k_i8, k_scale, _ = sage.sage_smooth_quant_k(to_dev(k), 64)
    q_i8, q_scale = sage.sage_quant_q(to_dev(q), w.sm_scale, 128)
    k_scale = k_scale * factor
    o, _ = sage.sage_attn_clock_debug(q_i8, q_scale, k_i8, k_scale, to_dev(v), causal=causal, block_q=128, block_k=64)
    ref = oracle.attn_l2(q_i8.cpu().numpy(), q_scale.cpu().numpy(), k_i8.cpu().numpy(), k_scale.cpu().numpy(), v, causal, 128, 64)
    assert_output_close(o.cpu().numpy(), ref, f"x {factor}")
