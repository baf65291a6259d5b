"""Softmax scales at the ends of what the calls accept: every finite positive one.

Scores of a huge scale are exact where the code products are powers of two: the query codes are 127 on a channel that
no key has, and 64 on a channel on which the keys have +-64 (their largest code, 127, is on a channel that no query
has).  Every product is then +-4096 and the result is known: a row takes the mean of the values of the positive keys it
sees, or of all keys it sees if none is positive."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
from gpu_util import sage

pytestmark = pytest.mark.gpu


def powers_of_two(B, H, N, D, seed):
    """q, k, v, and the result under a causal mask; the keys' mean is zero and the first half of them is negative."""
    rng = np.random.default_rng(seed)
    q = np.zeros((B, H, N, D), np.float16)
    q[..., 2], q[..., 1] = 127.0, 64.0
    sign = np.where(np.arange(N) < N // 2, -1.0, 1.0)
    k = np.zeros((B, H, N, D), np.float16)
    k[..., 0], k[..., 1] = 127.0 * sign, 64.0 * sign
    v = rng.standard_normal((B, H, N, D)).astype(np.float16)
    total = np.cumsum(v.astype(np.float64), axis=2)
    count = np.arange(1, N + 1)
    count[N // 2:] -= N // 2
    total[:, :, N // 2:] -= total[:, :, N // 2 - 1:N // 2].copy()
    return q, k, v, total / count[:, None]


@pytest.mark.parametrize("B, H, N, D, sm_scale", [
    (1, 2, 76, 64, 1e27), (1, 2, 130, 64, 1e27), (1, 2, 300, 64, 1e27), (1, 2, 200, 64, 1e30),      # one and two wavefronts per tile
    (30, 9, 200, 64, 1e27), (1, 2, 76, 128, 1e27), (1, 2, 256, 128, 1e30), (1, 2, 700, 64, 1e27)])   # more than a workgroup per CU; longer
def test_rows_whose_scores_are_all_far_below_zero(B, H, N, D, sm_scale):
    q, k, v, want = powers_of_two(B, H, N, D, 1700 + N + D)
    o = sage.sageattn(*(torch.from_numpy(x).cuda() for x in (q, k, v)), True, sm_scale, 1, 1)
    got = o.cpu().numpy().astype(np.float64)
    # weights are 0 and 1: half a unit of the fp16 result, and the fp32 sum of up to N values and its division (N 2^-24)
    assert np.isfinite(got).all()
    assert (np.abs(got - want) <= 2.0 ** -11 * np.abs(want) + 2.0 ** -25 + N * 2.0 ** -24 * np.abs(v).max()).all()


@pytest.mark.parametrize("N, D, block_k, sm_scale", [(200, 64, 64, 4e30), (300, 64, 1, 1e33), (200, 128, 64, 1e33), (130, 128, 1, 4e30)])
def test_huge_scales_with_the_int8_second_product(N, D, block_k, sm_scale):
    q, k, v, want = powers_of_two(1, 2, N, D, 1750 + N + D)
    o = sage.sageattn(*(torch.from_numpy(x).cuda() for x in (q, k, v)), True, sm_scale, 64 if block_k > 1 else 1, block_k, pv_int8=True)
    got = o.cpu().numpy().astype(np.float64)
    # the codes of V are half a step of their channel's scale off at most, a mean of them no more
    assert np.isfinite(got).all()
    step = np.abs(v.astype(np.float64)).max(axis=2, keepdims=True) / 127.0
    assert (np.abs(got - want) <= 0.5 * step + 2.0 ** -11 * np.abs(want) + 2.0 ** -25 + N * 2.0 ** -24 * np.abs(v).max()).all()


# every kernel that quantizes the queries itself: short sequences with one and two wavefronts per query tile, the attention
# kernel whole and in chunks of the keys, few queries, INT8 second product whole and in chunks
TINY = [(1, 2, 130, 130, 64, False, 128, 64, False), (3, 90, 200, 200, 64, True, 1, 1, False), (1, 2, 300, 300, 64, False, 64, 64, False),
        (1, 2, 400, 400, 64, True, 1, 1, False), (1, 2, 200, 200, 128, True, 128, 128, False),
        (1, 2, 700, 700, 64, True, 128, 64, False), (1, 2, 300, 300, 128, False, 32, 64, False), (2, 2, 100, 3000, 128, True, 64, 1, False),
        (1, 2, 1, 3000, 64, True, 128, 64, False), (1, 3, 20, 3000, 128, True, 1, 1, False),
        (1, 2, 300, 300, 64, True, 128, 64, True), (1, 2, 300, 300, 128, False, 64, 1, True), (1, 2, 20, 3000, 128, True, 128, 64, True)]


@pytest.mark.parametrize("sm_scale", [1e-38, 1e-41])
@pytest.mark.parametrize("B, H, Nq, Nkv, D, causal, bq, bk, pv8", TINY)
def test_scales_so_small_that_their_reciprocal_overflows(B, H, Nq, Nkv, D, causal, bq, bk, pv8, sm_scale):
    """127 / amax is infinite and the codes are clamped to their range.  They do not show: every score is nothing, and a row takes
    the mean of what it sees."""
    rng = np.random.default_rng(1790 + Nq + D)
    q, k, v = (rng.standard_normal((B, H, n, D)).astype(np.float16) for n in (Nq, Nkv, Nkv))
    q[:, :, 0, 3] = 0.0           # 0 times infinity
    v += np.float16(1.0)
    o = sage.sageattn(*(torch.from_numpy(x).cuda() for x in (q, k, v)), causal, sm_scale, bq, bk, pv_int8=pv8)
    got = o.cpu().numpy().astype(np.float64)
    v64 = v.astype(np.float64)
    seen = np.arange(Nkv - Nq, Nkv) + 1 if causal else np.full(Nq, Nkv)
    want = np.cumsum(v64, axis=2)[:, :, seen - 1] / seen[:, None]
    # all weights are equal: half a unit of the fp16 result (of the partial results too, where there are chunks) and the fp32
    # sums; half a step of the values' codes where the second product is INT8, whose weights are all 127
    bound = 2.0 ** -10 * np.abs(v64).max() + Nkv * 2.0 ** -24 * np.abs(v64).max()
    if pv8:
        bound = bound + 0.5 * np.abs(v64).max(axis=2, keepdims=True) / 127.0
    assert np.isfinite(got).all() and (np.abs(got - want) <= bound).all(), np.abs(got - want).max()
