"""sage_attention_fwd / sageattn() (the whole pass in one call) against the CPU oracle, at the sizes where its
plan changes or a tile ends: one token, edges of 32-row wavefronts, 64-key tiles and 128-row workgroups, the
limits of the single-launch path, different lengths, every granularity, both second products."""
import numpy as np
import pytest
import torch

import oracle
import paper_2410_02367_amd as sage
import sage_inputs as si
from gpu_util import ABS_TOL, assert_output_close, to_dev

pytestmark = pytest.mark.gpu

# B, H, Nq, Nkv, D, causal, block_q, block_k
CASES = [
    (1, 1, 1, 1, 64, True, 128, 64),
    (2, 3, 31, 31, 128, False, 128, 64),
    (1, 2, 33, 33, 64, True, 32, 64),
    (2, 2, 64, 64, 128, True, 64, 128),
    (1, 3, 129, 129, 128, True, 128, 64),
    (2, 2, 197, 197, 64, False, 128, 64),
    (1, 2, 256, 256, 64, False, 64, 64),
    (1, 2, 256, 256, 128, True, 128, 128),
    (2, 1, 257, 257, 128, False, 128, 64),
    (1, 2, 300, 300, 64, True, 1, 1),
    (1, 2, 200, 200, 128, False, 1, 1),
    (1, 2, 150, 150, 128, True, 1, 64),
    (1, 2, 250, 250, 64, False, 128, 1),
    (2, 2, 512, 512, 64, True, 128, 64),
    (1, 2, 513, 513, 128, True, 64, 64),
    (1, 3, 1105, 1105, 64, False, 128, 64),
    (1, 2, 1409, 1409, 128, True, 32, 128),
    (1, 2, 77, 200, 64, False, 128, 64),
    (1, 2, 700, 77, 128, False, 128, 64),
    (1, 2, 40, 256, 128, True, 128, 64),
    (1, 2, 130, 500, 64, True, 64, 64),
    (1, 2, 5, 1500, 128, True, 128, 64),
]


def inputs(i, B, H, Nq, Nkv, D):
    w = si.custom(f"fwd{i}", B, H, max(Nq, Nkv), D, False, 128, 64, k_noise=1.0, k_bias=3.0, seed=si.BASE_SEED + 900 + i)
    q, k, v = si.full(w)
    return np.ascontiguousarray(q[:, :, :Nq]), np.ascontiguousarray(k[:, :, :Nkv]), np.ascontiguousarray(v[:, :, :Nkv]), w.sm_scale


@pytest.mark.parametrize("i", range(len(CASES)))
def test_whole_pass_matches_the_oracle(i):
    B, H, Nq, Nkv, D, causal, bq, bk = CASES[i]
    print(f"[case] B{B} H{H} Nq{Nq} Nkv{Nkv} D{D} causal={causal} scales {bq}x{bk}", flush=True)
    q, k, v, sm = inputs(i, B, H, Nq, Nkv, D)
    need = sage.sage_attention_workspace(B, H, Nq, Nkv, D, causal, bq, bk)
    ws = torch.full((max(need, 1),), 0xFF, dtype=torch.uint8, device="cuda")      # contents on entry are ignored
    out = torch.full((B, H, Nq, D), float("nan"), dtype=torch.float16, device="cuda")
    sage.sage_attention_fwd(to_dev(q), to_dev(k), to_dev(v), causal, sm, bq, bk, out=out, workspace=ws)
    torch.cuda.synchronize()
    kq, ks, _ = oracle.smooth_quant_k(k, bk)
    qq, qs = oracle.quant_q(q, sm, bq)
    lq, lk = max(bq, 64) if bq != 1 else 128, max(bk, 64) if bk != 1 else 64
    ref = oracle.attn_l2_cross(qq, qs, kq, ks, v, causal, lq, lk, gran_q=bq, gran_k=bk)
    assert_output_close(out.cpu().numpy(), ref, f"case {i}")
    if Nq == Nkv:
        o8 = sage.sageattn(to_dev(q), to_dev(k), to_dev(v), causal, sm, bq, bk, pv_int8=True)
        torch.cuda.synchronize()
        vq, vs = oracle.quant_v(v)
        ref8, l_ref = oracle.attn_pv8(qq, qs, kq, ks, vq, vs, causal, 128, 64, gran_q=bq, gran_k=bk, return_l=True)
        # a code of P~ on the edge may fall either way: two codes of one key at most (small outputs: no share is asked)
        diff = np.abs(o8.cpu().numpy().astype(np.float64) - ref8.astype(np.float64))
        assert np.all(diff <= ABS_TOL + 2.0 * vs[:, :, None, :] / l_ref[..., None]), float(diff.max())


def test_mismatched_tensors_are_refused_before_any_launch():
    q = torch.zeros(1, 2, 64, 64, dtype=torch.float16, device="cuda")
    with pytest.raises(ValueError):
        sage.sageattn(q, q[:, :1].contiguous(), q[:, :1].contiguous())
    with pytest.raises(TypeError):
        sage.sageattn(q, q, q[:, :, :32].contiguous())
    with pytest.raises(TypeError):
        sage.sageattn(q, q.float(), q)
    with pytest.raises(TypeError):
        sage.sageattn(q.transpose(1, 2), q.transpose(1, 2), q.transpose(1, 2))
    with pytest.raises(sage.SageError):
        sage.sageattn(q, q, q, block_k=32)


# ------------------------------------------------------------------ launches that fill the chip

def on_device(seed, slabs, Nq, Nkv, D):
    g = torch.Generator(device="cuda").manual_seed(seed)

    def normal(n):
        return torch.randn((1, slabs, n, D), generator=g, device="cuda")

    return normal(Nq).half(), (normal(Nkv) + 3.0 * normal(1)).half(), normal(Nkv).half()


def oracle_slab(q, k, v, slab, causal, bq, bk):
    q, k, v = (np.ascontiguousarray(x[:, slab:slab + 1].cpu().numpy()) for x in (q, k, v))
    kq, ks, _ = oracle.smooth_quant_k(k, bk)
    qq, qs = oracle.quant_q(q, sage.sage_default_sm_scale(q.shape[3]), bq)
    lq, lk = max(bq, 64) if bq != 1 else 128, max(bk, 64) if bk != 1 else 64
    return oracle.attn_l2_cross(qq, qs, kq, ks, v, causal, lq, lk, gran_q=bq, gran_k=bk)


# Launches of 256-row workgroups: D = 128, at least 512 of them, more than 2048 keys (4096 with a mask), and without a mask
# no poorly filled last round: 128 x 17 of them are 8.5 rounds of the 256 compute units.
LARGE = [(128, 4100, False, 128, 64), (128, 4100, False, 64, 128), (128, 4100, False, 1, 64), (32, 16384, True, 128, 64),
         (128, 4100, False, 1, 1), (128, 4100, False, 32, 1), (32, 4200, True, 1, 1)]


@pytest.mark.parametrize("slabs,N,causal,bq,bk", LARGE)
def test_whole_pass_in_256_row_workgroups(slabs, N, causal, bq, bk):
    """Queries quantized inside the kernel (two 128-row scale blocks, four of 64 or one per row in a workgroup) give bit for
    bit what the separate calls give, on every row; the oracle's rows on one slab, where that is quick."""
    D = 128
    assert slabs * -(-N // 256) >= 512
    print(f"[case] {slabs} x {N} x {D} causal={causal} scales {bq}x{bk}", flush=True)
    q, k, v = on_device(N + bq, slabs, N, N, D)
    sm = sage.sage_default_sm_scale(D)
    o = sage.sageattn(q, k, v, causal, sm, bq, bk)
    q_i8, q_scale, k_i8, k_scale, _ = sage.sage_quant_qk(q, k, sm, bq, bk)
    chain = sage.sage_attn_fwd(q_i8, q_scale, k_i8, k_scale, v, causal, sm, bq, bk)
    torch.cuda.synchronize()
    assert torch.equal(o.view(torch.int16), chain.view(torch.int16))
    if N < 5000:
        assert_output_close(o[:, slabs - 1:].cpu().numpy(), oracle_slab(q, k, v, slabs - 1, causal, bq, bk))


# No mask, D = 128, more than 2048 keys: 128-row workgroups where their last round over 512 places is at most half full
# and they need at most six, else 256-row ones.  Slabs and rows on both sides of either line.
ROUNDS = [(8, 4096, False), (9, 3700, True), (3, 2049, True), (27, 2400, False), (40, 2432, True), (150, 2300, True), (171, 2300, False)]


@pytest.mark.parametrize("slabs,N,per_token", ROUNDS)
def test_workgroup_shape_by_its_last_round(slabs, N, per_token):
    D, (bq, bk) = 128, (1, 1) if per_token else (128, 64)
    tiles = slabs * -(-N // 128)
    print(f"[case] {slabs} x {N} x {D} scales {bq}x{bk}: {tiles} tiles, last round {(tiles - 1) % 512 + 1}", flush=True)
    q, k, v = on_device(slabs + N, slabs, N, N, D)
    o = sage.sageattn(q, k, v, False, sage.sage_default_sm_scale(D), bq, bk)
    torch.cuda.synchronize()
    assert_output_close(o[:, slabs - 1:].cpu().numpy(), oracle_slab(q, k, v, slabs - 1, False, bq, bk))


# The one-launch path with fewer workgroups than query tiles: each makes several turns (the next rows requested
# during the present ones, the scale words alternating).  Slabs x turns: 128-row workgroups, three (D = 64) or two per CU;
# 256-row ones, one per CU.
TURNS = [(768, 197, 197, 64, False, 128, 64, 2), (800, 400, 120, 64, False, 64, 1, 4), (520, 300, 100, 128, False, 128, 64, 3),
         (520, 128, 128, 128, True, 32, 64, 1), (300, 700, 500, 64, False, 128, 128, 3), (300, 512, 512, 64, True, 128, 64, 2),
         (260, 600, 256, 128, False, 1, 1, 3), (140, 1000, 256, 128, False, 128, 64, 4)]


@pytest.mark.parametrize("slabs,Nq,Nkv,D,causal,bq,bk,turns", TURNS)
def test_short_sequences_in_several_turns(slabs, Nq, Nkv, D, causal, bq, bk, turns):
    rows, per_cu = (256, 1) if Nkv * D > 16384 else (128, 3 if D == 64 else 2)
    groups = min(max(256 * per_cu // slabs, 1), -(-Nq // rows))
    assert sage.sage_attention_workspace(1, slabs, Nq, Nkv, D, causal, bq, bk) == 0 and -(-(-(-Nq // rows)) // groups) == turns
    print(f"[case] {slabs} x {Nq} x {Nkv} x {D} causal={causal} scales {bq}x{bk}", flush=True)
    q, k, v = on_device(Nq + Nkv, slabs, Nq, Nkv, D)
    sm = sage.sage_default_sm_scale(D)
    o = sage.sageattn(q, k, v, causal, sm, bq, bk)
    q_i8, q_scale, k_i8, k_scale, _ = sage.sage_quant_qk(q, k, sm, bq, bk)
    chain = sage.sage_attn_cross_fwd(q_i8, q_scale, k_i8, k_scale, v, causal, sm, bq, bk)
    torch.cuda.synchronize()
    # the separate calls add in another order: every row within the tolerance of either against the oracle
    assert bool(torch.isfinite(o).all()) and float((o.float() - chain.float()).abs().max()) <= ABS_TOL
    for slab in (0, slabs // 2, slabs - 1):
        assert_output_close(o[:, slab:slab + 1].cpu().numpy(), oracle_slab(q, k, v, slab, causal, bq, bk), f"slab {slab}")


# Two wavefronts per query tile, each with every other key tile: D = 64, 193 .. 512 keys and no more 128-row workgroups than
# CUs (half as many with a mask).  Odd and even numbers of tiles, a last half tile, rows that see no key of the second
# wavefront (causal rows 0 .. 63), fewer and more queries than keys, both sides of the line.
PAIRS = [(1, 193, 193, False, 64, 64), (3, 256, 256, True, 128, 128), (2, 257, 257, True, 1, 1), (5, 1, 500, True, 128, 64),
         (2, 200, 512, True, 32, 1), (2, 1000, 225, False, 128, 64), (64, 512, 512, False, 128, 64), (65, 512, 512, False, 64, 64),
         (64, 250, 250, True, 128, 64), (65, 250, 250, True, 1, 64)]


@pytest.mark.parametrize("slabs,Nq,Nkv,causal,bq,bk", PAIRS)
def test_short_sequences_with_two_wavefronts_per_query_tile(slabs, Nq, Nkv, causal, bq, bk):
    print(f"[case] {slabs} x {Nq} x {Nkv} x 64 causal={causal} scales {bq}x{bk}", flush=True)
    q, k, v = on_device(Nq + Nkv + bq, slabs, Nq, Nkv, 64)
    out = torch.full_like(q, float("nan"))
    sage.sage_attention_fwd(q, k, v, causal, sage.sage_default_sm_scale(64), bq, bk, out=out)
    torch.cuda.synchronize()
    for slab in (0, slabs - 1):
        assert_output_close(out[:, slab:slab + 1].cpu().numpy(), oracle_slab(q, k, v, slab, causal, bq, bk), f"slab {slab}")
