"""Performance cases of the library: what a program that uses it has it do, through its public entry points.

The three operations are attention forward (``attn_fwd``), the bf16 matrix product (``gemm_bf16``) and the FP8
mixture-of-experts feed-forward (``moe_ffn_fp8``).  The listed cases are points of the ranges that ``draw`` covers:
prefill from short prompts to a 32k context, a chunk of a prompt against a longer cache, head dimension 64,
decoding for one sequence and for a batch, linear layers in prefill and in decoding, products whose sizes are no
multiples of anything, and experts in prefill and in decoding.

Outputs are allocated by the entry points, as their defaults do; the expert layer's workspace is kept by the
program, as its interface asks for.
"""
from __future__ import annotations

import math

import torch

from paper_2604_18616_amd import attn_fwd, gemm_bf16, moe_ffn_fp8, moe_workspace_bytes

# Expert layers: model dimension, intermediate dimension, experts on this GPU, choices per token, ranks the experts
# are spread over (a token's choice is local with probability 1 / ep).
EXPERT_LAYERS = (
    (7168, 2048, 32, 4, 8),
    (4096, 14336, 8, 2, 1),
    (2048, 1408, 64, 6, 1),
    (2048, 768, 128, 8, 1),
)


def _attn(B, Hq, Hkv, Sq, Sk, D, causal, layout="bhsd", cache=0, k_shift=False):
    """layout: "bhsd" contiguous tensors, "bshd" views of [batch, sequence, head, d] buffers; cache: rows of the
    buffers that K and V are the first Sk rows of (0: exactly Sk)."""
    return dict(op="attn", B=B, Hq=Hq, Hkv=Hkv, Sq=Sq, Sk=Sk, D=D, causal=causal, layout=layout,
                cache=max(cache, Sk), k_shift=k_shift)


def _gemm(M, N, K, b_is_nk):
    return dict(op="gemm", M=M, N=N, K=K, b_is_nk=b_is_nk)


def _moe(T, layer):
    H, I, E, KTOP, EP = EXPERT_LAYERS[layer]
    return dict(op="moe", T=T, H=H, I=I, E=E, KTOP=KTOP, EP=EP)


def listed():
    return [
        # prefill of four prompts, grouped-query heads: the headline configuration of the benchmark
        dict(_attn(4, 32, 8, 4096, 4096, 128, True), name="attn_prefill_4k"),
        # prefill of one long context, the longest configuration of the benchmark
        dict(_attn(1, 32, 8, 32768, 32768, 128, True), name="attn_prefill_32k"),
        # a batch of short prompts on one GPU's share of the heads under tensor parallelism
        dict(_attn(16, 8, 1, 1024, 1024, 128, True), name="attn_prefill_1k"),
        # chunked prefill: 512 new tokens of two prompts against a cache that is longer and ends anywhere
        dict(_attn(2, 32, 8, 512, 5000, 128, True, layout="bshd", cache=8192), name="attn_chunk"),
        # bidirectional attention with head dimension 64 and shifted keys (benchmark configuration)
        dict(_attn(2, 16, 16, 8192, 8192, 64, False, k_shift=True), name="attn_d64"),
        # one decoding step of a batch against its caches
        dict(_attn(32, 32, 8, 1, 4096, 128, False, layout="bshd", cache=4608), name="attn_decode_batch"),
        # one decoding step of a single sequence: the smallest call, latency counts
        dict(_attn(1, 32, 8, 1, 2000, 128, False), name="attn_decode_single"),
        # the benchmark's square product; the arithmetic of a large linear layer
        dict(_gemm(8192, 8192, 8192, False), name="gemm_square_8k"),
        # a linear layer (weight stored [out, in]) while a batch of 16 decodes
        dict(_gemm(16, 14336, 4096, True), name="gemm_decode"),
        # sizes that are no multiples of anything
        dict(_gemm(999, 2001, 1501, False), name="gemm_odd"),
        # experts in prefill, the largest token count of the benchmark
        dict(_moe(16384, 0), name="moe_prefill"),
        # experts while a batch of 64 decodes
        dict(_moe(64, 0), name="moe_decode"),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _largest(key):
    return max(work(c)[key] for c in listed())


def draw(rng):
    """One more case of the ranges that the listed ones stand for."""
    max_flops, max_bytes = _largest("flops"), _largest("bytes")
    while True:
        case = _draw_any(rng)
        w = work(case)
        if w["flops"] <= max_flops and w["bytes"] <= max_bytes:
            return case


def _draw_heads(rng):
    """Query heads and kv heads: equal, grouped, or many on one."""
    hkv = rng.choice((1, 2, 4, 8, 16))
    return hkv * rng.choice((1, 2, 4, 8)), hkv


def _draw_any(rng):
    kind = rng.choice(("prefill", "chunk", "decode", "decode", "gemm", "linear", "odd", "moe", "moe"))
    layout = rng.choice(("bhsd", "bshd"))
    D = rng.choice((64, 128, 128))
    if kind == "prefill":
        hq, hkv = _draw_heads(rng)
        s = _log_int(rng, 128, 32768)
        s = rng.choice((s, s // 64 * 64))
        return _attn(_log_int(rng, 1, max(1, 65536 // s)), hq, hkv, s, s, D, rng.random() < 0.7, layout)
    if kind == "chunk":
        hq, hkv = _draw_heads(rng)
        sq = _log_int(rng, 16, 2048)
        sk = sq + _log_int(rng, 128, 16384)
        return _attn(_log_int(rng, 1, 8), hq, hkv, sq, sk, D, True, layout, cache=rng.choice((0, (sk + 1023) // 1024 * 1024)))
    if kind == "decode":
        hq, hkv = _draw_heads(rng)
        sk = _log_int(rng, 64, 65536)
        sq = rng.choice((1, 1, 1, 4))                        # one token, or a few speculated ones
        return _attn(_log_int(rng, 1, max(1, min(128, (1 << 18) // sk))), hq, hkv, sq, sk, D, sq > 1, layout,
                     cache=rng.choice((0, (sk + 255) // 256 * 256)))
    if kind == "gemm":                                      # multiples of 8, square and not
        m, n, k = (8 * _log_int(rng, 32, 1280) for _ in range(3))
        return _gemm(m, n, k, rng.random() < 0.5)
    if kind == "linear":                                    # few rows, a weight stored [out, in]
        return _gemm(_log_int(rng, 1, 128), 128 * _log_int(rng, 8, 224), 128 * _log_int(rng, 8, 112), True)
    if kind == "odd":
        return _gemm(_log_int(rng, 33, 2500), _log_int(rng, 33, 2500), _log_int(rng, 33, 2500), rng.random() < 0.5)
    layer = rng.choice((0, 0, 1, 2, 3))
    return _moe(_log_int(rng, 1, 16384 if layer == 0 else 8192), layer)


# ---------------------------------------------------------------------------------------------------------------
# preparation
# ---------------------------------------------------------------------------------------------------------------
def _normal(gen, shape):
    return torch.randn(shape, generator=gen, device="cuda", dtype=torch.bfloat16)


def _prepare_attn(c, gen):
    B, D = c["B"], c["D"]

    def rows(heads, seq, length):
        if c["layout"] == "bshd":
            return _normal(gen, (B, length, heads, D))[:, :seq].transpose(1, 2)
        return _normal(gen, (B, heads, length, D))[:, :, :seq]

    q = rows(c["Hq"], c["Sq"], c["Sq"])
    k, v = rows(c["Hkv"], c["Sk"], c["cache"]), rows(c["Hkv"], c["Sk"], c["cache"])
    if c["k_shift"]:                                        # a constant per kv head, half the spread: queries of a bounded norm
        q.mul_(0.5), k.mul_(0.5), v.mul_(0.5)
        k.add_(_normal(gen, (1, c["Hkv"], 1, 1)))
    return dict(q=q, k=k, v=v, causal=c["causal"])


def _prepare_gemm(c, gen):
    a = _normal(gen, (c["M"], c["K"]))
    b = _normal(gen, (c["N"], c["K"]) if c["b_is_nk"] else (c["K"], c["N"]))
    return dict(a=a, b=b, b_is_nk=c["b_is_nk"])


def _e4m3_weights(gen, shape):
    """Codes of 64 * N(0, 1), made one expert at a time."""
    out = torch.empty(shape, dtype=torch.uint8, device="cuda")
    for e in range(shape[0]):
        v = torch.randn(shape[1:], generator=gen, device="cuda", dtype=torch.bfloat16).mul_(64.0).clamp_(-448.0, 448.0)
        out[e] = v.to(torch.float8_e4m3fn).view(torch.uint8)
    return out


def _prepare_moe(c, gen):
    T, H, I, E, K = c["T"], c["H"], c["I"], c["E"], c["KTOP"]
    x = _normal(gen, (T, H))
    # each token chooses K distinct experts of all ranks; those of other ranks are marked -1 here
    chosen = torch.rand((T, E * c["EP"]), generator=gen, device="cuda").topk(K, dim=1).indices
    ids = torch.where(chosen < E, chosen, torch.full_like(chosen, -1)).to(torch.int32)
    wts = torch.rand((T, K), generator=gen, device="cuda") + 0.25
    wts = (wts / wts.sum(dim=1, keepdim=True)).contiguous()

    def scales(shape, fan_in):                              # unit-variance activations all the way
        return (1.0 + 0.25 * torch.rand(shape, generator=gen, device="cuda")) / (64.0 * math.sqrt(fan_in))

    w13, w2 = _e4m3_weights(gen, (E, 2 * I, H)), _e4m3_weights(gen, (E, H, I))
    s13, s2 = scales((E, 2 * I // 128, H // 128), H), scales((E, H // 128, I // 128), I)
    workspace = torch.empty(moe_workspace_bytes(T, H, I, E, K), dtype=torch.uint8, device="cuda")
    return dict(x=x, ids=ids, wts=wts, w13=w13, s13=s13, w2=w2, s2=s2, workspace=workspace)


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    make = {"attn": _prepare_attn, "gemm": _prepare_gemm, "moe": _prepare_moe}[case["op"]]
    return case["op"], make(case, gen)


# ---------------------------------------------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------------------------------------------
def run(state):
    op, s = state
    if op == "attn":
        return attn_fwd(s["q"], s["k"], s["v"], causal=s["causal"])
    if op == "gemm":
        return gemm_bf16(s["a"], s["b"], b_is_nk=s["b_is_nk"])
    return moe_ffn_fp8(s["x"], s["ids"], s["wts"], s["w13"], s["s13"], s["w2"], s["s2"], workspace=s["workspace"])


def work(case):
    c = case
    if c["op"] == "attn":
        pairs = c["Sq"] * c["Sk"]
        if c["causal"]:                                     # the last query sees every key, each one before it one fewer
            seen = min(c["Sq"], c["Sk"])
            pairs = seen * c["Sk"] - seen * (seen - 1) // 2
        q_rows, kv_rows = c["B"] * c["Hq"] * c["Sq"], c["B"] * c["Hkv"] * c["Sk"]
        return {"bytes": 4.0 * c["D"] * (q_rows + kv_rows) + 4.0 * q_rows, "flops": 4.0 * c["D"] * c["B"] * c["Hq"] * pairs}
    if c["op"] == "gemm":
        M, N, K = c["M"], c["N"], c["K"]
        return {"bytes": 2.0 * (M * K + K * N + M * N), "flops": 2.0 * M * N * K}
    T, H, I, E, K, total = c["T"], c["H"], c["I"], c["E"], c["KTOP"], c["E"] * c["EP"]
    # expected counts: a token reaches a given expert with probability K / total
    used = E * (1.0 - (1.0 - K / total) ** T)
    pairs = T * K / c["EP"]
    return {"bytes": 4.0 * T * H + 3.0 * H * I * used * (1.0 + 4.0 / 16384) + 8.0 * T * K, "flops": 6.0 * H * I * pairs}


# Measured on the listed cases against the same definitions in 64 bits (2-norm, largest difference): attention, with
# its probabilities rounded to bf16 in front of the second product and a bf16 result, 2.4e-3 and 0.04; the matrix
# product, one rounding to bf16, 1.7e-3 and 3.9e-3; the expert layer, whose intermediate is e4m3, where a sum that
# comes out an ulp apart flips a code, 2.1e-3 and 0.1.  About four times that:
_TOLERANCE = {
    "attn": {"rel": 1e-2, "max": 0.16},
    "gemm": {"rel": 7e-3, "max": 0.016},
    "moe": {"rel": 8e-3, "max": 0.4},
}


def tolerance(case):
    return dict(_TOLERANCE[case["op"]])


# ---------------------------------------------------------------------------------------------------------------
# the same results in 64 bits
# ---------------------------------------------------------------------------------------------------------------
def _exact_attn(c, s):
    B, Hq, Hkv, Sq, Sk, D = (c[k] for k in ("B", "Hq", "Hkv", "Sq", "Sk", "D"))
    o = torch.empty((B, Hq, Sq, D), dtype=torch.float64, device="cuda")
    lse = torch.empty((B, Hq, Sq), dtype=torch.float64, device="cuda")
    rows = max(1, min(Sq, (1 << 28) // Sk))                 # 2 GiB of scores at a time
    keys = torch.arange(Sk, device="cuda")
    for b in range(B):
        for hk in range(Hkv):
            kt, v = s["k"][b, hk].double().t().contiguous(), s["v"][b, hk].double()
            for h in range(hk * (Hq // Hkv), (hk + 1) * (Hq // Hkv)):
                for i in range(0, Sq, rows):
                    scores = (s["q"][b, h, i:i + rows].double() * float(D) ** -0.5) @ kt
                    if c["causal"]:
                        last = torch.arange(i, i + scores.shape[0], device="cuda") + (Sk - Sq)
                        scores.masked_fill_(keys[None, :] > last[:, None], -math.inf)
                    lse[b, h, i:i + rows] = total = torch.logsumexp(scores, dim=1)
                    o[b, h, i:i + rows] = scores.sub_(total[:, None]).exp_() @ v
    return o, lse


def _exact_gemm(c, s):
    b = s["b"].double()
    return s["a"].double() @ (b.t().contiguous() if c["b_is_nk"] else b)


def _groups_of_128(v):
    """e4m3 codes and a scale per 128 values, both decided in 32 bits as the format is defined, widened again."""
    g = v.float().reshape(v.shape[0], -1, 128)
    scale = g.abs().amax(dim=2, keepdim=True) * torch.tensor(1.0 / 448.0, device=v.device)
    scale = torch.where(scale > 0, scale, torch.ones_like(scale))
    codes = (g * (1.0 / scale)).clamp_(-448.0, 448.0).to(torch.float8_e4m3fn)
    return (codes.double() * scale.double()).reshape(v.shape)


def _widened(codes, scales):
    w = codes.view(torch.float8_e4m3fn).double()
    return w * scales.double().repeat_interleave(128, 0).repeat_interleave(128, 1)


def _exact_moe(c, s):
    T, H, I, E = c["T"], c["H"], c["I"], c["E"]
    y = torch.zeros((T, H), dtype=torch.float64, device="cuda")
    for e in range(E):
        tok, slot = (s["ids"] == e).nonzero(as_tuple=True)
        if tok.numel() == 0:
            continue
        xq = _groups_of_128(s["x"][tok])
        gu = xq @ _widened(s["w13"][e], s["s13"][e]).t().contiguous()
        gate, up = gu[:, :I], gu[:, I:]
        a = _groups_of_128(gate / (1.0 + torch.exp(-gate)) * up)
        rows = a @ _widened(s["w2"][e], s["s2"][e]).t().contiguous()
        y.index_add_(0, tok, rows * s["wts"][tok, slot].double()[:, None])
    return y


def exact(case, seed):
    """What run() returns for these inputs, in 64 bits; for the expert layer with the codes of its two quantizations,
    which are part of its definition.  None where that takes too long."""
    if case["op"] == "attn" and work(case)["flops"] > 1.2e13:
        return None
    op, s = prepare(case, seed)
    return {"attn": _exact_attn, "gemm": _exact_gemm, "moe": _exact_moe}[op](case, s)
