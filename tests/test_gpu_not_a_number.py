"""Inputs are finite by contract, but a NaN in a query or a value (a padding row that was never written) stays where it
is: the other query rows, the other channels and the rows that do not see the token come out as with zeros in its place, on
every path that finds the maxima itself.  (Up to rounding: a wavefront raises the running maxima of its rows together.)"""
import numpy as np
import pytest
import torch

import paper_2410_02367_amd as sage
import sage_inputs as si
from gpu_util import ABS_TOL, to_dev

pytestmark = pytest.mark.gpu

# B, H, Nq, Nkv, D, causal, block_q, pv_int8: one launch, 128-row and 256-row workgroups, few queries, INT8 second product
CASES = [
    (1, 2, 200, 200, 64, False, 128, False),
    (1, 2, 200, 200, 128, True, 64, False),
    (1, 2, 700, 700, 64, True, 128, False),
    (1, 3, 700, 700, 128, False, 32, False),
    (1, 2, 20, 700, 128, True, 128, False),
    (1, 2, 200, 200, 128, True, 128, True),
    (1, 2, 700, 700, 64, True, 128, True),
    (2, 2, 1300, 1300, 128, True, 1, True),
    (1, 32, 3900, 3900, 128, False, 128, False),
]


@pytest.mark.parametrize("i", range(len(CASES)))
def test_a_nan_stays_in_its_row(i):
    B, H, Nq, Nkv, D, causal, bq, pv8 = CASES[i]
    print(f"[case] B{B} H{H} Nq{Nq} Nkv{Nkv} D{D} causal={causal} block_q {bq} pv_int8={pv8}", flush=True)
    w = si.custom(f"nan{i}", B, H, max(Nq, Nkv), D, False, seed=si.BASE_SEED + 1500 + i)
    q, k, v = si.full(w)
    q, k, v = (np.ascontiguousarray(x) for x in (q[:, :, :Nq], k[:, :, :Nkv], v[:, :, :Nkv]))
    row, token, channel = 3, Nkv - 5, 7
    outs = []
    for value in (0.0, np.nan):
        qx, vx = q.copy(), v.copy()
        qx[:, :, row, :] = value
        if pv8:
            vx[:, :, token, channel] = value
        outs.append(sage.sageattn(to_dev(qx), to_dev(k), to_dev(vx), causal, w.sm_scale, bq, 64, pv_int8=pv8))
    torch.cuda.synchronize()
    zeros, nans = (o.float().cpu().numpy() for o in outs)
    fine = np.abs(zeros - nans) <= ABS_TOL          # false where either is not a number
    fine[:, :, row, :] = True
    if pv8:
        # the token's code of that channel may be any: for the rows that see it
        first = token - (Nkv - Nq) if causal else 0
        fine[:, :, max(first, 0):, channel] = True
    assert fine.all(), np.argwhere(~fine)[:5]


@pytest.mark.parametrize("i", range(len(CASES)))
def test_a_nan_gets_the_code_that_the_separate_calls_give_it(i):
    """A query that is no number has the code -127 wherever it is quantized: its row, whose other channels are finite, comes
    out of the whole pass as it does of the pre-pass calls and the attention call."""
    B, H, Nq, Nkv, D, causal, bq, pv8 = CASES[i]
    print(f"[case] B{B} H{H} Nq{Nq} Nkv{Nkv} D{D} causal={causal} block_q {bq} pv_int8={pv8}", flush=True)
    w = si.custom(f"nancode{i}", B, H, max(Nq, Nkv), D, False, seed=si.BASE_SEED + 1600 + i)
    q, k, v = (to_dev(np.ascontiguousarray(x[:, :, :n])) for x, n in zip(si.full(w), (Nq, Nkv, Nkv)))
    q[:, :, 3, 7] = float("nan")            # the lane's first channels and its last, in rows of either half of a wavefront's
    q[:, :, Nq - 1, D - 1] = float("nan")
    o = sage.sageattn(q, k, v, causal, w.sm_scale, bq, 64, pv_int8=pv8)
    q_i8, q_scale, k_i8, k_scale, _ = sage.sage_quant_qk(q, k, w.sm_scale, bq, 64)
    assert bool((q_i8[:, :, 3, 7] == -127).all()) and bool((q_i8[:, :, Nq - 1, D - 1] == -127).all())
    if pv8:
        chain = sage.sage_attn_pv_int8_cross_fwd(q_i8, q_scale, k_i8, k_scale, *sage.sage_quant_v(v), causal, w.sm_scale, bq, 64)
    else:
        chain = sage.sage_attn_cross_fwd(q_i8, q_scale, k_i8, k_scale, v, causal, w.sm_scale, bq, 64)
    torch.cuda.synchronize()
    assert bool(torch.isfinite(o).all()) and float((o.float() - chain.float()).abs().max()) <= ABS_TOL
