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


def flat(r):
    return r if isinstance(r, tuple) else (r,)


@pytest.mark.parametrize("handle", [False, True])
@pytest.mark.parametrize("what", ["attention", "attention_int8", "quant_qk", "quant_v", "rope_k", "split"])
def test_a_named_streams_scratch_is_not_handed_out_while_it_runs(what, handle):
    """The named stream is kept busy, so the call's kernels run after later work of the current stream has taken and
    filled memory of the same sizes: scratch and outputs must not be among it."""
    q, k = tensor(1, 4, 1500, 64), tensor(1, 4, 1500, 64)
    table = torch.ones(1500, 32, device="cuda")
    q_i8, q_scale, k_i8, k_scale, _ = sage.sage_quant_qk(q[:, :, :40].contiguous(), k, 0.125)
    calls = {
        "attention": lambda s: sage.sage_attention_fwd(q, k, q, True, 0.125, stream=s),
        "attention_int8": lambda s: sage.sage_attention_fwd(q, k, q, True, 0.125, pv_int8=True, stream=s),
        "quant_qk": lambda s: sage.sage_quant_qk(q, k, 0.125, stream=s),
        "quant_v": lambda s: sage.sage_quant_v(q, stream=s),
        "rope_k": lambda s: sage.sage_rope_smooth_quant_k(k, table, table, stream=s),
        "split": lambda s: sage.sage_attn_cross_split_fwd(q_i8, q_scale, k_i8, k_scale, k, True, 0.125, n_splits=4, stream=s),
    }
    expected = [t.cpu() for t in flat(calls[what](None))]
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        torch.cuda._sleep(5_000_000)
    got = flat(calls[what](side.cuda_stream if handle else side))
    junk = [torch.full((1 << n,), 0x55, dtype=torch.uint8, device="cuda") for n in range(9, 24) for _ in range(4)]
    torch.cuda.current_stream().wait_stream(side)
    for a, b in zip(got, expected):
        assert torch.equal(a.cpu(), b)
    assert all(int(x[-1]) == 0x55 for x in junk)
    # with every buffer given nothing is allocated, whatever the stream
    if what == "quant_v":
        ws = torch.empty(max(sage.sage_quant_v_workspace(1, 4, 1500, 64), 4) // 4, dtype=torch.int32, device="cuda")
        given = [torch.zeros_like(t) for t in got]
        torch.cuda.synchronize()
        back = sage.sage_quant_v(q, given[0], given[1], ws, stream=side)
        torch.cuda.synchronize()
        assert back[0] is given[0] and all(torch.equal(a.cpu(), b) for a, b in zip(given, expected))
