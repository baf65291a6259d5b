"""The kernel for at most 32 queries per slab and the merge of key chunks, where they can go wrong: 32 and 33
queries, fewer key tiles than wavefronts, a ragged last tile, rows that see no key of some tile, more slabs than
compute units, more chunks than one batch of the merge, more rows than its wavefront-per-row form takes."""
import numpy as np
import pytest
import torch

import oracle
import paper_2410_02367_amd as sage
import sage_inputs as si
from gpu_util import assert_output_close, to_dev

pytestmark = pytest.mark.gpu

# B, H, Nq, Nkv, D, causal, block_q, block_k, chunks
CASES = [
    (1, 2, 1, 1, 64, True, 128, 64, 1),
    (1, 2, 5, 31, 128, True, 128, 64, 1),
    (2, 2, 32, 33, 128, True, 64, 64, 1),
    (1, 3, 32, 32, 64, True, 128, 64, 1),
    (1, 2, 33, 200, 128, True, 128, 64, 1),
    (2, 2, 31, 97, 64, False, 32, 128, 1),
    (1, 3, 17, 289, 128, True, 1, 1, 1),
    (1, 2, 2, 161, 64, True, 128, 1, 1),
    (3, 90, 7, 300, 128, True, 128, 64, 1),
    (3, 90, 3, 270, 128, False, 1, 1, 1),
    (1, 2, 3, 6000, 128, True, 128, 64, 40),
    (2, 33, 64, 700, 64, False, 128, 64, 5),
    (2, 20, 110, 600, 128, True, 128, 64, 2),
]


@pytest.mark.parametrize("i", range(len(CASES)))
def test_few_queries(i):
    B, H, Nq, Nkv, D, causal, bq, bk, chunks = CASES[i]
    print(f"[case] B{B} H{H} Nq{Nq} Nkv{Nkv} D{D} causal={causal} scales {bq}x{bk} chunks {chunks}", flush=True)
    w = si.custom(f"few{i}", B, H, max(Nq, Nkv), D, False, k_noise=1.0, k_bias=3.0, seed=si.BASE_SEED + 1300 + i)
    q, k, v = si.full(w)
    q, k, v = (np.ascontiguousarray(x) for x in (q[:, :, :Nq], k[:, :, :Nkv], v[:, :, :Nkv]))
    kd, vd = to_dev(k), to_dev(v)
    k_i8, k_scale, _ = sage.sage_smooth_quant_k(kd, bk)
    q_i8, q_scale = sage.sage_quant_q(to_dev(q), w.sm_scale, bq)
    o = sage.sage_attn_cross_split_fwd(q_i8, q_scale, k_i8, k_scale, vd, causal, w.sm_scale, bq, bk, n_splits=chunks)
    torch.cuda.synchronize()
    qq, qs = oracle.quant_q(q, w.sm_scale, bq)
    kq, ks, _ = oracle.smooth_quant_k(k, bk)
    lq, lk = max(bq, 64) if bq != 1 else 128, max(bk, 64) if bk != 1 else 64
    ref = oracle.attn_l2_cross(qq, qs, kq, ks, v, causal, lq, lk, gran_q=bq, gran_k=bk)
    assert_output_close(o.cpu().numpy(), ref, f"case {i}")
