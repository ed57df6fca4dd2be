"""Performance cases of libdn: the calls a Transformer layer makes through this package.

Each case is one call of one entry point of ``paper_2502_17728_amd.ops`` with its inputs
and prepared weights already on the GPU, as a serving or encoding program holds them.
Sizes are those of the package's named workloads (BERT-base, 7B/8B-class and 70B-class
layers) and of the token counts and sequence lengths around them.

``kind`` selects the call:
  linear     ln_linear_deferred / rms_linear_deferred   x[M, K] . W[K, N]
  swiglu     rms_swiglu_deferred                        x[M, K] . W_gate, W_up[K, N]
  softmax    softmax_pv_deferred                        S[BH, L, L], V[BH, L, d]
  attention  attention_deferred                         Q[BH * g, Lq, d], K and V[BH, Lk, d]
  decode     attention_decode_deferred                  the same, Lq new tokens against the cache
"""
import math

import torch

from paper_2502_17728_amd import ops

DEV = "cuda:0"
EPS = 1e-5
DTYPE = {"f32": torch.float32, "bf16": torch.bfloat16}


def listed():
    return [
        # BERT-base encoder, LayerNorm -> FFN up-projection over one short text, fp32
        dict(name="ln_f32_bert_ffn", kind="linear", norm="layernorm", dtype="f32", M=128, K=768, N=3072),
        # BERT-base self-attention over 512 tokens, scores already formed
        dict(name="softmax_bert", kind="softmax", BH=12, L=512, d=64, causal=False),
        # one token of one sequence through the QKV projection of a 7B-class layer
        dict(name="ln_qkv_1_token", kind="linear", norm="layernorm", dtype="bf16", M=1, K=4096, N=12288),
        # eight sequences decoding together, gated MLP of a 70B-class layer
        dict(name="swiglu_8_tokens", kind="swiglu", dtype="bf16", M=8, K=8192, N=28672),
        # a hundred sequences decoding together (or a short prompt), QKV of a 7B-class layer
        dict(name="ln_qkv_100_tokens", kind="linear", norm="layernorm", dtype="bf16", M=100, K=4096, N=12288),
        # a ragged prefill chunk through the gated MLP of an 8B-class layer
        dict(name="swiglu_500_tokens", kind="swiglu", dtype="bf16", M=500, K=4096, N=14336),
        # a 4096-token prompt through the QKV projection of a 7B-class layer
        dict(name="ln_qkv_4096_tokens", kind="linear", norm="layernorm", dtype="bf16", M=4096, K=4096, N=12288),
        # an 8192-token prompt through the FFN up-projection of a 70B-class layer
        dict(name="ln_ffn_8192_tokens", kind="linear", norm="layernorm", dtype="bf16", M=8192, K=8192, N=28672),
        # causal self-attention over 8192 tokens from stored scores, 32 heads
        dict(name="softmax_causal_8192", kind="softmax", BH=32, L=8192, d=128, causal=True),
        # causal self-attention over an 8192-token prompt, 32 heads
        dict(name="attention_causal_8192", kind="attention", BH=32, g=1, Lq=8192, Lk=8192, d=128, causal=True),
        # a ragged 1000-token prompt in an 8B-class layer: 32 query heads over 8 key/value heads
        dict(name="attention_gqa_1000", kind="attention", BH=8, g=4, Lq=1000, Lk=1000, d=128, causal=True),
        # eight sequences decoding against a ragged cache, 32 query heads over 8 key/value heads each
        dict(name="decode_gqa_5001", kind="decode", BH=64, g=4, Lq=1, Lk=5001, d=128),
    ]


MAX_FLOPS = 2.0 * 8192 * 8192 * 28672  # the largest listed case
SHAPES = [(768, 2304), (768, 3072), (4096, 12288), (4096, 6144), (8192, 28672)]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _log8(rng, lo, hi):
    return max(8, _log(rng, lo, hi) // 8 * 8)


def _features(rng):
    """A hidden size and an output size: a layer's own or any other of the range (multiples of 8)."""
    if rng.random() < 0.6:
        return rng.choice(SHAPES)
    return _log8(rng, 512, 8192), _log8(rng, 1024, 28672)


def draw(rng):
    """One more case: sizes over the ranges the listed ones stand for, odd ones among them."""
    kind = rng.choice(["linear", "linear", "swiglu", "softmax", "attention", "decode"])
    d = rng.choice([64, 128, 128])
    if kind == "linear":
        dtype = rng.choice(["bf16", "bf16", "bf16", "f32"])
        K, N = _features(rng)
        M = _log(rng, 1, 1024 if dtype == "f32" else 8192)
        return dict(kind=kind, norm=rng.choice(["layernorm", "rms"]), dtype=dtype, M=M, K=K, N=N)
    if kind == "swiglu":
        K, N = rng.choice([(4096, 14336), (8192, 28672), (_log8(rng, 512, 8192), _log8(rng, 1024, 28672))])
        M = min(_log(rng, 1, 8192), int(MAX_FLOPS / (4.0 * K * N)))
        return dict(kind=kind, dtype="bf16", M=M, K=K, N=N)
    if kind == "softmax":
        L = _log8(rng, 64, 8192)
        return dict(kind=kind, BH=_log(rng, 8, 32), L=L, d=d, causal=rng.random() < 0.6)
    g = rng.choice([1, 4, 8])
    if kind == "attention":
        causal = rng.random() < 0.7
        Lk = _log(rng, 64, 8192)
        Lq = Lk if causal else _log(rng, 17, 8192)
        return dict(kind=kind, BH=max(1, _log(rng, 8, 32) // g), g=g, Lq=Lq, Lk=Lk, d=d, causal=causal)
    Lk = _log(rng, 128, 16384)
    return dict(kind=kind, BH=min(_log(rng, 4, 512), max(4, (256 << 20) // (Lk * d))), g=g,
                Lq=rng.choice([1, 1, 1, 2]), Lk=Lk, d=d)


# ------------------------------------------------------------------------------- inputs
def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed) * 7919 + 17)


def _normal(gen, shape, std=1.0, dtype=torch.bfloat16):
    t = torch.randn(shape, generator=gen, device=DEV, dtype=torch.float32)
    return (t * std if std != 1.0 else t).to(dtype)


def _rows(case, gen):
    """Activations: unit normal, and in the bf16 layers of 4096 features 8 outlier channels 20 times larger."""
    x = torch.randn((case["M"], case["K"]), generator=gen, device=DEV, dtype=torch.float32)
    if case["K"] == 4096:
        ch = torch.randperm(case["K"], generator=gen, device=DEV)[:8]
        x[:, ch] *= 20.0
    return x.to(DTYPE[case["dtype"]])


def _inputs(case, seed):
    gen, kind = _gen(seed), case["kind"]
    if kind in ("linear", "swiglu"):
        K, N, dt = case["K"], case["N"], DTYPE[case["dtype"]]
        t = dict(x=_rows(case, gen), gamma=(torch.rand(K, generator=gen, device=DEV) + 0.5).to(dt))
        for name in ("W",) if kind == "linear" else ("Wg", "Wu"):
            t[name] = _normal(gen, (K, N), K ** -0.5, dt)
        if case.get("norm") == "layernorm":
            t["beta"] = _normal(gen, (K,), math.sqrt(0.02), dt)
        return t
    if kind == "softmax":
        BH, L, d = case["BH"], case["L"], case["d"]
        S = torch.empty((BH, L, L), dtype=torch.bfloat16, device=DEV)
        above = torch.ones((L, L), dtype=torch.bool, device=DEV).triu(1) if case["causal"] else None
        for h in range(BH):  # the scores of unit-normal queries and keys
            q, k = _normal(gen, (L, d)).float(), _normal(gen, (L, d)).float()
            s = torch.matmul(q, k.t()) * (2.0 if above is None else 1.0) / math.sqrt(d)
            S[h] = (s if above is None else s.masked_fill(above, float("-inf"))).to(torch.bfloat16)
        return dict(S=S, V=_normal(gen, (BH, L, d)))
    kv = (case["BH"], case["Lk"], case["d"])
    return dict(Q=_normal(gen, (case["BH"] * case["g"], case["Lq"], case["d"])), K=_normal(gen, kv), V=_normal(gen, kv))


def prepare(case, seed):
    """The activations and, for the projections, the weights prepared once as a loaded model keeps them."""
    t, kind = _inputs(case, seed), case["kind"]
    if kind == "linear":
        w = ops.ln_linear_prepare(t["W"], t["gamma"], t.get("beta"))
        return dict(case=case, x=t["x"], w=w)
    if kind == "swiglu":
        return dict(case=case, x=t["x"], w=ops.swiglu_prepare(t["Wg"], t["Wu"], t["gamma"]))
    if kind == "decode":
        Lq = case["g"] * case["Lq"]
        n = ops.attention_decode_workspace_bytes(case["BH"], Lq, case["Lk"], case["d"])
        t["workspace"] = torch.empty(max(n, 16), dtype=torch.uint8, device=DEV)
    return dict(case=case, **t)


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "linear":
        call = ops.ln_linear_deferred if case["norm"] == "layernorm" else ops.rms_linear_deferred
        return call(state["x"], state["w"], EPS)
    if kind == "swiglu":
        return ops.rms_swiglu_deferred(state["x"], state["w"], EPS)
    if kind == "softmax":
        return ops.softmax_pv_deferred(state["S"], state["V"], causal=case["causal"])
    if kind == "attention":
        return ops.attention_deferred(state["Q"], state["K"], state["V"], causal=case["causal"])
    return ops.attention_decode_deferred(state["Q"], state["K"], state["V"], workspace=state["workspace"])


# ------------------------------------------------------------------------------- what is counted and compared
def work(case):
    kind = case["kind"]
    if kind in ("linear", "swiglu"):
        e = 4 if case["dtype"] == "f32" else 2
        M, K, N = case["M"], case["K"], case["N"]
        mats = 1 if kind == "linear" else 2
        return {"bytes": e * (M * K + mats * K * N + M * N), "flops": 2.0 * mats * M * K * N}
    d, BH = case["d"], case["BH"]
    if kind == "softmax":
        L = case["L"]
        pairs = BH * (L * (L + 1) // 2 if case["causal"] else L * L)
        return {"bytes": 2 * (pairs + 2 * BH * L * d), "flops": 2.0 * pairs * d}
    Lq, Lk, g = case["Lq"], case["Lk"], case["g"]
    pairs = BH * g * (Lk * (Lk + 1) // 2 if case.get("causal") else Lq * Lk)
    return {"bytes": 2 * (2 * BH * g * Lq * d + 2 * BH * Lk * d), "flops": 4.0 * pairs * d}


def tolerance(case):
    """About four times the error measured against 64 bits.  bf16 weights, numerators and outputs round
    once each (2^-9 relative): 2.0e-3 to 2.4e-3 off, 2.9e-3 where two products meet; fp32: 5e-7 over
    768 products, growing with the square root of their number to about 1.5e-6 over 8192."""
    if case.get("dtype") == "f32":
        return {"rel": 6e-6}
    return {"rel": 1.2e-2 if case["kind"] == "swiglu" else 1e-2}


def exact(case, seed):
    t, kind = _inputs(case, seed), case["kind"]
    f64 = torch.float64
    if kind in ("linear", "swiglu"):
        x = t["x"].to(f64)
        if case.get("norm") == "layernorm":
            x = x - x.mean(1, keepdim=True)
        y = x / torch.sqrt((x * x).mean(1, keepdim=True) + EPS) * t["gamma"].to(f64)
        if "beta" in t:
            y = y + t["beta"].to(f64)
        if kind == "linear":
            return torch.matmul(y, t["W"].to(f64))
        g = torch.matmul(y, t["Wg"].to(f64))
        return g * torch.sigmoid(g) * torch.matmul(y, t["Wu"].to(f64))
    if kind == "softmax":
        heads = []
        for h in range(case["BH"]):
            s = t["S"][h].to(f64)
            if case["causal"]:
                s = s.masked_fill(torch.ones_like(s, dtype=torch.bool).triu(1), float("-inf"))
            heads.append(torch.matmul(torch.softmax(s, 1), t["V"][h].to(f64)))
        return torch.stack(heads)
    heads = []
    for h in range(case["BH"] * case["g"]):
        kh = h // case["g"]
        s = torch.matmul(t["Q"][h].to(f64), t["K"][kh].to(f64).t().contiguous()) / math.sqrt(case["d"])
        if case.get("causal"):
            s = s.masked_fill(torch.ones_like(s, dtype=torch.bool).triu(1), float("-inf"))
        heads.append(torch.matmul(torch.softmax(s, 1), t["V"][kh].to(f64)))
    return torch.stack(heads)
