"""What the FP16 weights of a row keep when one key carries most of it, and what a row may depend on.

A dominant key in the first tile (the attention sink of a language model) leaves the other keys with weights of 2^-20 and
less; a small value there and a common one elsewhere make the result the share of all the others.  Keys that a causal row does
not see must not reach it, not even through their scale.  And O and l must be sums of the same weights: values of one
everywhere give a result of exactly one."""
import math

import numpy as np
import pytest
import torch

import paper_2410_02367_amd as sage
from gpu_util import assert_output_close, bits

pytestmark = pytest.mark.gpu


def softmax_of_codes(qq, qs, kq, ks, v, causal=False):
    """Attention of one slab over codes and scales (one per row and key) in 64 bits."""
    s = (qq.double() @ kq.double().T) * qs.double()[:, None] * ks.double()[None, :]
    if causal:
        s = s.masked_fill(torch.ones_like(s, dtype=torch.bool).triu(1), -math.inf)
    return torch.softmax(s, dim=1) @ v.double()


# slabs, N, D, block_k, n_splits; 160 queries.  128-row workgroups with one set of wavefronts are D = 64 with more than 256 of
# them or with the keys in chunks.
SINKS = [(1, 131072, 64, 64, 1), (1, 131072, 64, 128, 2), (130, 16384, 64, 64, 1), (1, 131072, 128, 64, 1), (2, 16384, 128, 128, 1),
         (1, 131072, 128, 64, 8), (2, 16384, 128, 1, 1), (1, 16384, 64, 1, 1)]


@pytest.mark.parametrize("where", ["first tile", "middle"])
@pytest.mark.parametrize("slabs,N,D,block_k,n_splits", SINKS)
def test_the_tail_beside_a_dominant_key(slabs, N, D, block_k, n_splits, where):
    """The tail's share p = 3 % (N = 131072) or 1 % (16384) is held by N keys with weights between 2^-21 and 2^-24 of the
    dominant one.  FP16 rounds those to multiples of 2^-24, unbiased over scores that vary by e^0.5: the share is right to
    well within the tolerance; weights scaled down by another 2^4 are lost, and with them all of p."""
    print(f"[case] {slabs} x 160 against {N} x {D}, keys scaled per {block_k}, {n_splits} chunks, dominant key in the {where}", flush=True)
    share, std, Nq = 0.97 if N > 16384 else 0.99, 0.5, 160
    rng = np.random.default_rng(2 * N + D + block_k)
    at = 5 if where == "first tile" else N // 2 + 7
    kq = np.clip(np.rint(40.0 * rng.standard_normal((N, D))), -127, 127)
    qq = np.clip(np.rint(40.0 * rng.standard_normal((Nq, D))), -127, 127)
    kq[:, 0], qq[:, 0] = 0, 127
    unit = std / (40.0 * 40.0 * math.sqrt(D - 1))
    ks = np.full(-(-N // block_k), unit, np.float32)
    gain = (math.log(N) + std ** 2 / 2 + math.log(share / (1 - share))) / (127.0 * 127.0 * unit)
    b = at // block_k
    ks[b] *= gain
    rows = slice(b * block_k, (b + 1) * block_k)
    kq[rows] = np.rint(kq[rows] / gain)
    kq[at] = 0
    kq[at, 0] = 127
    v = np.ones((N, D)) + 0.1 * rng.standard_normal((N, D))
    v[at] = 0
    dev = lambda x, t: torch.from_numpy(x).to(t).cuda()
    qd, kd, vd, ksd = dev(qq, torch.int8), dev(kq, torch.int8), dev(v, torch.float16), dev(ks, torch.float32)
    qs = torch.ones(-(-Nq // 128), dtype=torch.float32, device="cuda")
    per_slab = lambda x: x.expand(1, slabs, *x.shape).contiguous()
    args = [per_slab(x) for x in (qd, qs, kd, ksd, vd)]
    if n_splits == 1:
        out = sage.sage_attn_cross_fwd(*args, False, D ** -0.5, 128, block_k)
    else:
        out = sage.sage_attn_cross_split_fwd(*args, False, D ** -0.5, 128, block_k, n_splits=n_splits)
    ref = softmax_of_codes(qd, qs.repeat_interleave(128)[:Nq], kd, ksd.repeat_interleave(block_k)[:N], vd).cpu().numpy()
    out = out.cpu().numpy()
    for s in {0, slabs - 1}:
        assert_output_close(out[0, s], ref, f"slab {s}")


# slabs, N, D, block_k: two sets of wavefronts, one set at D = 64, and at D = 128 workgroups of 128 and of 256 rows
CAUSAL = [(2, 1024, 64, 64), (65, 577, 64, 64), (2, 960, 128, 128), (2, 1024, 128, 64), (17, 2100, 128, 64)]


@pytest.mark.parametrize("factor", [1e3, 1e5, 1e20])
@pytest.mark.parametrize("slabs,N,D,block_k", CAUSAL)
def test_rows_do_not_depend_on_the_scale_of_keys_they_do_not_see(slabs, N, D, block_k, factor):
    print(f"[case] {slabs} x {N} x {D} causal, last block of {block_k} keys x {factor}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(N + D)
    normal = lambda: torch.randn((1, slabs, N, D), generator=gen, device="cuda").half()
    q, k, v = normal(), normal(), normal()
    sm = D ** -0.5
    k_i8, k_scale, _ = sage.sage_smooth_quant_k(k, block_k)
    q_i8, q_scale = sage.sage_quant_q(q, sm, 128)
    before = sage.sage_attn_fwd(q_i8, q_scale, k_i8, k_scale, v, True, sm, 128, block_k)
    k_scale[..., -1] *= factor
    after = sage.sage_attn_fwd(q_i8, q_scale, k_i8, k_scale, v, True, sm, 128, block_k)
    first = (N - 1) // block_k * block_k          # a multiple of the 32 rows of a wavefront
    a, b = (x[:, :, :first].cpu().numpy() for x in (before, after))
    assert np.isfinite(a).all()
    assert np.array_equal(bits(a), bits(b))


@pytest.mark.parametrize("block_k", [1, 64])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("slabs", [2, 150])
def test_the_denominator_sums_the_weights_that_multiply_the_values(slabs, D, block_k):
    """64 equal weights wait for their product when the second tile's one visible key raises the maximum by 0.8 to 1 in the
    exponent (one row in 32 by 10, which makes the wavefront raise).  A factor of 2^-0.8 to 2^-1 is rounded by up to 2^-12,
    relatively 2^-11; where the sum held other weights than the product, rows would come out as 1 - 2^-11."""
    print(f"[case] {slabs} x 256 against 1088 x {D}, keys scaled per {block_k}", flush=True)
    Nq, N = 256, 1088
    qq = torch.zeros((1, slabs, Nq, D), dtype=torch.int8)
    qq[..., 0] = 127
    qq[..., 1] = 100
    step = torch.linspace(0.8, 1.0, Nq)
    step[5::32] = 10.0
    kq = torch.zeros((1, slabs, N, D), dtype=torch.int8)
    kq[:, :, 65:, 0] = -127
    kq[:, :, 64, 1] = 100
    qs = (step * math.log(2.0) / 1e4).expand(1, slabs, Nq).contiguous()      # one scale per query; the visible key's score is step ln 2
    ks = torch.ones((1, slabs, -(-N // block_k)))
    if block_k == 1:
        ks[:, :, 65:] = 100.0
        kq[:, :, 65:, 0] = -127
    else:
        # one scale per block: the other keys of the second one are as low as its scale lets them be, 2^-1.3 to 2^-16
        ks[:, :, 2:] = 100.0
    v = torch.ones((1, slabs, N, D), dtype=torch.float16)
    out = sage.sage_attn_cross_fwd(qq.cuda(), qs.cuda(), kq.cuda(), ks.cuda(), v.cuda(), False, D ** -0.5, 1, block_k)
    assert (out.cpu() == 1.0).all()


# slabs, N, D, block_q, block_k, n_splits (0: the whole call, which quantizes the queries in the kernel): workgroups of either
# shape, one and two sets of wavefronts, keys in chunks, scales that differ within a wavefront, one scale per key
COARSE = [(2, 1024, 64, 128, 64, 1), (40, 1000, 64, 128, 128, 1), (2, 1024, 64, 128, 64, 3), (2, 1024, 128, 128, 64, 1), (17, 2100, 128, 128, 128, 1),
          (2, 1000, 128, 128, 64, 4), (2, 1024, 64, 1, 64, 1), (40, 1000, 64, 32, 64, 1), (2, 1000, 128, 1, 128, 1), (2, 1100, 64, 128, 64, 0),
          (40, 1000, 64, 1, 64, 0), (2, 700, 128, 64, 64, 0), (2, 1024, 64, 1, 1, 1), (2, 1024, 128, 1, 1, 1)]


@pytest.mark.parametrize("q_large,k_large", [(60.0, -60000.0), (100.0, 60000.0), (731.0, -4321.0), (3000.0, 50000.0)])
@pytest.mark.parametrize("where", ["first", "middle", "last"])
@pytest.mark.parametrize("slabs,N,D,block_q,block_k,n_splits", COARSE)
def test_scales_that_make_one_unit_of_a_score_a_range_of_weights(slabs, N, D, block_q, block_k, n_splits, where, q_large, k_large):
    """One channel of a key and of every 16th query is so large that one unit of an integer score is 2^24 to 2^1700 in the weights:
    the maximum of a row cannot lie on a grid of such units, neither in that tile nor in the ones before and after it."""
    print(f"[case] {slabs} x {N} x {D}, scales {block_q}x{block_k}, {n_splits} chunks, {where} key {k_large}, queries {q_large}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(N + D)
    normal = lambda: torch.randn((1, slabs, N, D), generator=gen, device="cuda")
    q, k, v = normal(), normal(), normal().clamp(-1.99, 1.99).half()
    q[:, :, ::16, 3] = q_large
    k[:, :, {"first": 0, "middle": N // 2 + 1, "last": N - 1}[where], 3] = k_large
    sm = D ** -0.5
    k_i8, k_scale, _ = sage.sage_smooth_quant_k(k.half(), block_k)
    q_i8, q_scale = sage.sage_quant_q(q.half(), sm, block_q)
    if n_splits == 0:
        out = sage.sageattn(q.half(), k.half(), v, False, sm, block_q, block_k)
    elif n_splits == 1:
        out = sage.sage_attn_fwd(q_i8, q_scale, k_i8, k_scale, v, False, sm, block_q, block_k)
    else:
        out = sage.sage_attn_cross_split_fwd(q_i8, q_scale, k_i8, k_scale, v, False, sm, block_q, block_k, n_splits=n_splits)
    for s in {0, slabs - 1}:
        qs, ks = q_scale[0, s].repeat_interleave(block_q)[:N], k_scale[0, s].repeat_interleave(block_k)[:N]
        assert block_k == 1 or float((qs.max() * ks.max()) * math.log2(math.e)) > 24
        ref = softmax_of_codes(q_i8[0, s], qs, k_i8[0, s], ks, v[0, s]).cpu().numpy()
        assert_output_close(out[0, s].cpu().numpy(), ref, f"slab {s}")


# slabs, N, D, block_q, block_k, causal: short sequences, one and two wavefronts per query tile
SHORT = [(500, 200, 64, 128, 64, False), (500, 197, 64, 128, 128, True), (2, 256, 64, 128, 64, False), (2, 400, 64, 64, 128, True), (3, 97, 64, 64, 64, False),
         (2, 256, 128, 128, 64, False), (300, 250, 128, 64, 64, True), (2, 256, 64, 1, 1, False), (300, 255, 128, 1, 1, True)]


@pytest.mark.parametrize("q_large,k_large", [(60.0, -60000.0), (100.0, 60000.0), (3000.0, 50000.0), (3000.0, -50000.0)])
@pytest.mark.parametrize("where", ["first", "middle", "last"])
@pytest.mark.parametrize("slabs,N,D,block_q,block_k,causal", SHORT)
def test_such_scales_in_short_sequences(slabs, N, D, block_q, block_k, causal, where, q_large, k_large):
    print(f"[case] {slabs} x {N} x {D} causal={causal}, scales {block_q}x{block_k}, {where} key {k_large}, queries {q_large}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(N + D)
    normal = lambda: torch.randn((1, slabs, N, D), generator=gen, device="cuda")
    q, k, v = normal(), normal(), normal().clamp(-1.99, 1.99).half()
    q[:, :, ::16, 3] = q_large
    k[:, :, {"first": 0, "middle": N // 2 + 1, "last": N - 1}[where], 3] = k_large
    q, k, sm = q.half(), k.half(), D ** -0.5
    out = sage.sageattn(q, k, v, causal, sm, block_q, block_k)
    k_i8, k_scale, _ = sage.sage_smooth_quant_k(k, block_k)
    q_i8, q_scale = sage.sage_quant_q(q, sm, block_q)
    for s in {0, slabs - 1}:
        qs, ks = q_scale[0, s].repeat_interleave(block_q)[:N], k_scale[0, s].repeat_interleave(block_k)[:N]
        ref = softmax_of_codes(q_i8[0, s], qs, k_i8[0, s], ks, v[0, s], causal).cpu().numpy()
        assert_output_close(out[0, s].cpu().numpy(), ref, f"slab {s}")
