"""What the Python wrappers refuse, with tensors on the device (host tensors never reach the native half)."""
import pytest
import torch

import paper_2410_02367_amd as sage

pytestmark = pytest.mark.gpu


def tensor(*shape):
    return torch.randn(shape, generator=torch.Generator().manual_seed(5)).half().cuda()


@pytest.mark.parametrize("missing", ["both", "cos", "sin"])
def test_rope_calls_refuse_missing_tables(missing):
    """Without its tables a RoPE call is an error, never the call without a rotation."""
    x = tensor(1, 2, 96, 64)
    table = torch.ones(96, 32, device="cuda")
    cos, sin = (None if missing in ("both", name) else table for name in ("cos", "sin"))
    with pytest.raises((AttributeError, TypeError)):
        sage.sage_rope_quant_q(x, cos, sin, 0.125)
    with pytest.raises((AttributeError, TypeError)):
        sage.sage_rope_smooth_quant_k(x, cos, sin)
    assert sage.sage_rope_quant_q(x, table, table, 0.125)[0].shape == x.shape


@pytest.mark.parametrize("v_given", ["fp16", "codes"])
def test_int8_second_product_refuses_calls_without_its_scales(v_given):
    """fp16 values without scales are an error for the INT8 second product, never the FP16 one's input."""
    x = tensor(1, 2, 128, 64)
    q_i8, q_scale = sage.sage_quant_q(x, 0.125)
    k_i8, k_scale, _ = sage.sage_smooth_quant_k(x)
    v = x if v_given == "fp16" else sage.sage_quant_v(x)[0]
    for call in (sage.sage_attn_pv_int8_fwd, sage.sage_attn_pv_int8_cross_fwd, sage.sage_attn_pv_int8_cross_split_fwd):
        with pytest.raises(TypeError):
            call(q_i8, q_scale, k_i8, k_scale, v, None, False, 0.125)
