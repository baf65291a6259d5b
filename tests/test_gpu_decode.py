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


# More workgroups than compute units at D = 128: two wavefronts each (short ones), four (more than 2048 keys), or the
# general kernel (fewer than 384 workgroups of at least 1280 keys, one scale per block).
MANY = [(300, 1279, 128, 64), (300, 1280, 128, 64), (383, 1300, 128, 64), (384, 1300, 128, 64), (300, 1300, 1, 1),
        (400, 2048, 128, 64), (400, 2049, 128, 64), (257, 2100, 1, 1), (90, 4000, 128, 64)]


@pytest.mark.parametrize("slabs,Nkv,bq,bk", MANY)
def test_few_queries_of_many_slabs(slabs, Nkv, bq, bk):
    D, Nq = 128, 3
    n = sage.sage_attn_split_count(1, slabs, Nq, Nkv, True, 0)
    print(f"[case] {slabs} x ({Nq}, {Nkv}) x {D} scales {bq}x{bk} chunks {n}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(slabs + Nkv)
    q, v = (torch.randn((1, slabs, m, D), generator=g, device="cuda").half() for m in (Nq, Nkv))
    k = (torch.randn((1, slabs, Nkv, D), generator=g, device="cuda") + 3.0 * torch.randn((1, slabs, 1, D), generator=g, device="cuda")).half()
    sm = sage.sage_default_sm_scale(D)
    q_i8, q_scale, k_i8, k_scale, _ = sage.sage_quant_qk(q, k, sm, bq, bk)
    outs = [sage.sage_attn_cross_split_fwd(q_i8, q_scale, k_i8, k_scale, v, True, sm, bq, bk),
            sage.sage_attn_cross_fwd(q_i8, q_scale, k_i8, k_scale, v, True, sm, bq, bk),
            sage.sageattn(q, k, v, True, sm, bq, bk)]
    torch.cuda.synchronize()
    for slab in (0, 131 % slabs, slabs - 1):
        a, b, c = (np.ascontiguousarray(x[:, slab:slab + 1].cpu().numpy()) for x in (q, k, v))
        qq, qs = oracle.quant_q(a, sm, bq)
        kq, ks, _ = oracle.smooth_quant_k(b, bk)
        ref = oracle.attn_l2_cross(qq, qs, kq, ks, c, True, 128, 64, gran_q=bq, gran_k=bk)
        for o in outs:
            assert_output_close(o[:, slab:slab + 1].cpu().numpy(), ref, f"slab {slab}")
