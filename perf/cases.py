"""The attention calls that programs make of this library, as cases whose speed can be measured.

A case is a dict of plain values:
  kind     "attention"  the whole of sageattn() on fp16 Q, K, V (equal lengths, or Nq queries against Nkv keys)
           "rope"       a language model's layer: RoPE fused into both pre-pass calls, then the attention call
           "cached"     serving: K (and, with pv_int8, V) were quantized when they entered the cache, the call
                        quantizes the new queries and attends to the cache; buffers are the server's own
  B, H, Nq, Nkv, D      shape; causal: the mask, aligned at the end of the keys
  block_q, block_k      tokens per quantization scale (1: per token)
  pv_int8               second product in INT8 instead of FP16
  k_noise, k_bias       K = k_noise N(0,1) + a bias per channel ~ N(0, k_bias^2), shared by all tokens of a head
  outliers              one channel of every head of K is eight times larger
"""
import math

import torch

import paper_2410_02367_amd as sage


def _case(name, kind, B, H, Nq, Nkv, D, causal, block_q=128, block_k=64, pv_int8=False, k_noise=0.5, k_bias=3.0,
          outliers=False):
    c = {"kind": kind, "B": B, "H": H, "Nq": Nq, "Nkv": Nkv, "D": D, "causal": causal, "block_q": block_q, "block_k": block_k,
         "pv_int8": pv_int8, "k_noise": k_noise, "k_bias": k_bias, "outliers": outliers}
    return c if name is None else dict(c, name=name)


def listed():
    return [
        # one small call, as in a test or a little model: launches and the host are all of it
        _case("tiny_256", "attention", 1, 2, 256, 256, 64, False, block_q=64),
        # a vision transformer's layer: many heads, a length that no tile divides
        _case("vit_197", "attention", 12, 64, 197, 197, 64, False),
        # image generation at low resolution
        _case("image_1105", "attention", 4, 24, 1105, 1105, 64, False),
        # a language model on short prompts, batched
        _case("llm_1536", "attention", 4, 32, 1536, 1536, 128, True, k_noise=1.0, k_bias=4.0),
        # image generation at high resolution
        _case("image_4096", "attention", 4, 32, 4096, 4096, 128, False),
        # video generation: long, not causal, ragged
        _case("video_17776", "attention", 2, 30, 17776, 17776, 64, False),
        # a language model's prefill of a long prompt
        _case("prefill_16k", "attention", 1, 32, 16384, 16384, 128, True, k_noise=1.0, k_bias=4.0, outliers=True),
        # the same with the INT8 second product
        _case("prefill_16k_int8", "attention", 1, 32, 16384, 16384, 128, True, pv_int8=True, k_noise=1.0, k_bias=4.0, outliers=True),
        # prefill of a whole book, a share of the heads per GPU
        _case("prefill_128k", "attention", 1, 8, 131072, 131072, 128, True, k_noise=1.0, k_bias=4.0),
        # a language model's layer with one scale per token and RoPE in the pre-pass
        _case("rope_token_4096", "rope", 2, 32, 4096, 4096, 128, True, block_q=1, block_k=1, k_noise=1.0, k_bias=4.0),
        # decoding: one new token against a cache of 16K
        _case("decode_16k", "cached", 1, 32, 1, 16384, 128, True, k_noise=1.0, k_bias=4.0, outliers=True),
        # chunked prefill: the next 512 tokens of a prompt against the cache
        _case("chunk_512_of_16k", "cached", 1, 32, 512, 16384, 128, True, k_noise=1.0, k_bias=4.0, outliers=True),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["attention"] * 6 + ["cross"] * 2 + ["rope"] * 2 + ["cached"] * 3)
    D = rng.choice([64, 128])
    slabs = _log_uniform(rng, 2, 800)
    H = min(slabs, rng.randint(2, 40))
    B = max(1, slabs // H)
    # at most the tensors of prefill_128k and half of its arithmetic
    longest = int(min(65536, 2 ** 27 / (B * H * D), math.sqrt(8e12 / (4.0 * B * H * D))))
    N = _log_uniform(rng, 64, longest)
    causal = rng.random() < 0.5
    per_token = rng.random() < 0.2
    block_q, block_k = (1, 1) if per_token else (rng.choice([128, 128, 64]), rng.choice([64, 64, 128]))
    pv_int8 = kind != "rope" and rng.random() < 0.25
    Nq = N
    if kind == "cross":
        # a short side against a long one: text against an image, or the other way round
        Nq, causal = min(longest, _log_uniform(rng, 32, 8192)), False
        kind = "attention"
    elif kind == "cached":
        # from one new token to a chunk of a prompt
        N = _log_uniform(rng, min(1024, longest), longest)
        Nq, causal = min(N, _log_uniform(rng, 1, 1024)), True
    noise, bias = rng.choice([(0.5, 3.0), (1.0, 4.0)])
    return _case(None, kind, B, H, Nq, N, D, causal, block_q, block_k, pv_int8, noise, bias, rng.random() < 0.25)


def _scale(case):
    return sage.sage_default_sm_scale(case["D"])


def prepare(case, seed):
    B, H, Nq, Nkv, D = (case[n] for n in ("B", "H", "Nq", "Nkv", "D"))
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)

    def normal(*shape):
        return torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32)

    q = normal(B, H, Nq, D).half()
    v = normal(B, H, Nkv, D).half()
    k = normal(B, H, Nkv, D).mul_(case["k_noise"]).add_(normal(B, H, 1, D).mul_(case["k_bias"]))
    if case["outliers"]:
        channel = torch.randint(D, (B, H, 1, 1), generator=gen, device="cuda").expand(B, H, Nkv, 1)
        k.scatter_(3, channel, k.gather(3, channel).mul_(8.0))
    state = {"case": case, "q": q, "k": k.half(), "v": v, "sm_scale": _scale(case)}
    if case["kind"] == "rope":
        # the tables a model makes once: base 10000, position t
        inv = 10000.0 ** (-torch.arange(0, D, 2, device="cuda", dtype=torch.float64) / D)
        angle = torch.arange(Nkv, device="cuda", dtype=torch.float64)[:, None] * inv[None, :]
        state["cos"], state["sin"] = angle.cos().float(), angle.sin().float()
    elif case["kind"] == "cached":
        k_i8, k_scale, _ = sage.sage_smooth_quant_k(state.pop("k"), case["block_k"])
        state["k_i8"], state["k_scale"] = k_i8, k_scale
        if case["pv_int8"]:
            state["v_i8t"], state["v_scale"] = sage.sage_quant_v(state.pop("v"))
        nbq = -(-Nq // case["block_q"])
        state["q_i8"] = torch.empty((B, H, Nq, D), dtype=torch.int8, device="cuda")
        state["q_scale"] = torch.empty((B, H, nbq), dtype=torch.float32, device="cuda")
        state["out"] = torch.empty((B, H, Nq, D), dtype=torch.float16, device="cuda")
        need = sage.sage_attn_split_workspace(B, H, Nq, Nkv, D, case["causal"])
        state["workspace"] = torch.empty(max(need, 16), dtype=torch.uint8, device="cuda")
    return state


def run(state):
    case, sm_scale = state["case"], state["sm_scale"]
    bq, bk, causal = case["block_q"], case["block_k"], case["causal"]
    if case["kind"] == "attention":
        return sage.sageattn(state["q"], state["k"], state["v"], causal=causal, sm_scale=sm_scale, block_q=bq, block_k=bk,
                             pv_int8=case["pv_int8"])
    if case["kind"] == "rope":
        q_i8, q_scale = sage.sage_rope_quant_q(state["q"], state["cos"], state["sin"], sm_scale, bq)
        k_i8, k_scale, k_mean = sage.sage_rope_smooth_quant_k(state["k"], state["cos"], state["sin"], bk)
        out = sage.sage_attn_fwd(q_i8, q_scale, k_i8, k_scale, state["v"], causal, sm_scale, bq, bk)
        return {"q_i8": q_i8, "q_scale": q_scale, "k_i8": k_i8, "k_scale": k_scale, "k_mean": k_mean, "out": out}
    sage.sage_quant_q(state["q"], sm_scale, bq, q_i8=state["q_i8"], q_scale=state["q_scale"])
    if case["pv_int8"]:
        out = sage.sage_attn_pv_int8_cross_split_fwd(state["q_i8"], state["q_scale"], state["k_i8"], state["k_scale"],
                                                     state["v_i8t"], state["v_scale"], causal, sm_scale, bq, bk,
                                                     out=state["out"], workspace=state["workspace"])
    else:
        out = sage.sage_attn_cross_split_fwd(state["q_i8"], state["q_scale"], state["k_i8"], state["k_scale"], state["v"],
                                             causal, sm_scale, bq, bk, out=state["out"], workspace=state["workspace"])
    return {"q_i8": state["q_i8"], "q_scale": state["q_scale"], "out": out}


def work(case):
    """Each input read once, each output written once; the two products over the visible (query, key) pairs."""
    slabs, Nq, Nkv, D = case["B"] * case["H"], case["Nq"], case["Nkv"], case["D"]
    pairs = Nq * Nkv - (Nq * (Nq - 1) // 2 if case["causal"] else 0)
    q, kv, scales = slabs * Nq * D, slabs * Nkv * D, 4 * slabs * (-(-Nq // case["block_q"]))
    key_scales = 4 * slabs * (-(-Nkv // case["block_k"]))
    if case["kind"] == "cached":
        moved = 2 * q + q + scales + kv + key_scales + (kv if case["pv_int8"] else 2 * kv) + 2 * q
    elif case["kind"] == "rope":
        moved = 2 * q + 4 * kv + 2 * 4 * Nkv * (D // 2) + q + scales + kv + key_scales + 4 * slabs * D + 2 * q
    else:
        moved = 2 * q + 4 * kv + 2 * q
    return {"bytes": moved, "flops": 4 * slabs * pairs * D}


def tolerance(case):
    """FP16 results of FP16 weights: half a unit of 2^-10 each.  "max" is for single values near zero, whose error is that
    of the large values they are a difference of (the first rows of a causal mask average few keys, the rms is that of the
    last ones).  With the INT8 second product a weight on the edge of two codes may take either: one code of one key."""
    if case["pv_int8"]:
        return {"rel": 4e-3, "max": 0.9}
    return {"rel": 1e-3, "max": 0.2}
