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
