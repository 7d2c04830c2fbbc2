"""Cases for timing the library: what programs that use it have it do, through ``paper_2505_20839_amd.binding``.

The sizes are those of the repository's own workloads (Llama2-7B: hidden 4096, FFN 11008; Llama3-8B: hidden
4096, FFN 14336, fused QKV width 6144, 8 key/value heads of 128 with 4 query heads each), at token counts from
one decode row to a long prefill, with uneven counts among them: a batch, a chunk or a cache has the length it
happens to have.  Values are drawn as in ``workloads.py`` (activations N(0,1) with 1 % of the columns x 20,
uniform INT4 codes, group scales U[0.005, 0.05] as E4M3, key/value scales U[0.02, 0.2]).

Kinds of case:
  linear     a whole layer from bf16 activations in one call (fq_w4a8_linear)
  residual   a layer whose output is added to the residual stream (fq_quantize_act + fq_w4a8_gemm_add)
  ffn        a feed-forward block: quantiser, gate/up with fused SiLU(gate) * up, down projection + residual
  block      the four linear layers of one decoder block at a decode batch, captured once into a HIP graph
             and replayed, as a serving loop runs them (the benchmark times its steps the same way)
  attention  the attention operands of one decode step on an INT4 key/value cache: scores, quantisation of the
             probabilities, output
  cache      packing the key and the value cache of prefilled sequences
  offline    a weight matrix from bf16 to the GEMM's operands: CAS, PTS, quantisation, packing
"""
import math

import torch

from paper_2505_20839_amd import binding as fq

GROUP = 128
SQRT_D = 128 ** -0.5


def listed():
    return [
        # one token of one sequence through a square projection: launch and host latency
        {"name": "token_proj", "kind": "linear", "M": 1, "N": 4096, "K": 4096},
        # sixteen sequences decoding: QKV, attention-output, gate/up and down layers, replayed from a graph
        {"name": "decode_block_16", "kind": "block", "M": 16, "hidden": 4096, "qkv": 6144, "ffn": 14336},
        # an uneven decode batch through the widest projection of a block
        {"name": "batch_37_up", "kind": "linear", "M": 37, "N": 14336, "K": 4096},
        # a short prefill chunk through the down projection, residual added in the epilogue
        {"name": "chunk_200_down", "kind": "residual", "M": 200, "N": 4096, "K": 11008},
        # a chunk of a chunked prefill through the up projection
        {"name": "chunk_500_up", "kind": "linear", "M": 500, "N": 14336, "K": 4096},
        # an uneven prompt through a whole feed-forward block
        {"name": "ffn_1000", "kind": "ffn", "M": 1000, "hidden": 4096, "ffn": 11008},
        # the benchmark's default workload: a prefill of 2048 tokens through one projection
        {"name": "prefill_2048", "kind": "linear", "M": 2048, "N": 11008, "K": 4096},
        # the largest configuration: 8192 tokens through the widest projection
        {"name": "prefill_8192", "kind": "linear", "M": 8192, "N": 14336, "K": 4096},
        # 32 sequences x 8 key/value heads with 4096 cached tokens each
        {"name": "attention_batch", "kind": "attention", "H": 256, "R": 4, "T": 4096},
        # one long sequence: few heads, a cache of a length that is a multiple of nothing
        {"name": "attention_long", "kind": "attention", "H": 8, "R": 4, "T": 32001},
        # 16 prefilled sequences' caches packed for decoding
        {"name": "cache_pack", "kind": "cache", "H": 128, "T": 2000},
        # a gate or up matrix quantised and packed, once per weight
        {"name": "offline_weights", "kind": "offline", "N": 11008, "K": 4096},
    ]


def _log_int(rng, lo, hi, step=1):
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return int(min(hi, max(lo, round(v / step) * step)))


def draw(rng):
    kind = rng.choice(["linear", "linear", "residual", "ffn", "block", "attention", "attention", "cache", "offline"])
    if kind in ("linear", "residual"):
        N = _log_int(rng, 1024, 22016, rng.choice([8, 32, 128]))
        K = _log_int(rng, 1024, 14336, GROUP)
        return {"kind": kind, "M": _log_int(rng, 1, min(8192, 8192 * 14336 * 4096 // (N * K))), "N": N, "K": K}
    if kind == "ffn":
        return {"kind": kind, "M": _log_int(rng, 1, 2500), "hidden": _log_int(rng, 2048, 5120, GROUP),
                "ffn": _log_int(rng, 5632, 14336, GROUP)}
    if kind == "block":
        return {"kind": kind, "M": _log_int(rng, 1, 64), "hidden": _log_int(rng, 2048, 5120, GROUP),
                "qkv": _log_int(rng, 3072, 12288, GROUP), "ffn": _log_int(rng, 5632, 14336, GROUP)}
    if kind == "attention":
        H = 8 * _log_int(rng, 1, 64)
        return {"kind": kind, "H": H, "R": _log_int(rng, 1, 16), "T": _log_int(rng, 200, min(32768, (1 << 21) // H))}
    if kind == "cache":
        H = 8 * _log_int(rng, 1, 64)
        return {"kind": kind, "H": H, "T": _log_int(rng, 200, min(32768, (1 << 19) // H))}
    return {"kind": kind, "N": _log_int(rng, 1024, 22016, 8), "K": _log_int(rng, 1024, 11008, GROUP)}


# ---- inputs -------------------------------------------------------------------------------------------------

def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed) * 7919 + 12345)


def _acts(g, M, K, scale=1.0):
    """bf16 activations: N(0,1), 1 % of the columns x 20."""
    x = torch.randn((M, K), generator=g, device="cuda")
    x[:, torch.randperm(K, generator=g, device="cuda")[: max(1, K // 100)]] *= 20.0
    return (x * scale).to(torch.bfloat16)


def _int4(g, *shape):
    return torch.randint(-8, 8, shape, generator=g, device="cuda", dtype=torch.int8)


def _e4m3(g, lo, hi, *shape):
    u = torch.rand(shape, generator=g, device="cuda") * (hi - lo) + lo
    return u.to(torch.float8_e4m3fn).view(torch.uint8)


def _layer(g, N, K, keep_codes):
    """(codes or packed weights, group scales) of an [N,K] layer."""
    q, gs = _int4(g, N, K), _e4m3(g, 0.005, 0.05, N, K // GROUP)
    return (q if keep_codes else fq.fq_pack_weights(q)), gs


def _inputs(case, seed, raw):
    """Everything a case starts from; `raw`: the INT4 codes of layers and caches instead of the packed forms."""
    g, kind, s = _gen(seed), case["kind"], {"case": case}
    if kind == "linear":
        M, N, K = case["M"], case["N"], case["K"]
        s["x"], s["w"] = _acts(g, M, K), _layer(g, N, K, raw)
    elif kind == "residual":
        M, N, K = case["M"], case["N"], case["K"]
        s["x"], s["w"] = _acts(g, M, K), _layer(g, N, K, raw)
        s["res"] = _acts(g, M, N, 16.0)
    elif kind == "ffn":
        M, D, F = case["M"], case["hidden"], case["ffn"]
        s["x"], s["res"] = _acts(g, M, D), _acts(g, M, D, 16.0)
        s["gu"], s["down"] = _layer(g, 2 * F, D, raw), _layer(g, D, F, raw)
    elif kind == "block":
        M, D, Q, F = case["M"], case["hidden"], case["qkv"], case["ffn"]
        s["x"], s["attn"], s["res"] = _acts(g, M, D), _acts(g, M, D), _acts(g, M, D, 16.0)
        s["qkv"], s["o"] = _layer(g, Q, D, raw), _layer(g, D, D, raw)
        s["gu"], s["down"] = _layer(g, 2 * F, D, raw), _layer(g, D, F, raw)
    elif kind == "attention":
        H, R, T = case["H"], case["R"], case["T"]
        Qb = torch.randn((H * R, GROUP), generator=g, device="cuda").to(torch.bfloat16)
        ldp = (T + 15) // 16 * 16                             # probability rows padded with zeros to whole 16-byte steps
        logits = 2.0 * torch.randn((H * R, T), generator=g, device="cuda")
        s["p"] = torch.nn.functional.pad(torch.softmax(logits, dim=1), (0, ldp - T)).to(torch.bfloat16)
        k, v = _int4(g, H, T, GROUP), _int4(g, H, T, GROUP)
        s["ks"], s["vs"] = _e4m3(g, 0.02, 0.2, H, T), _e4m3(g, 0.02, 0.2, H, T)
        if raw:
            s["q"], s["k"], s["v"] = Qb, k, v
        else:
            qc, qs = fq.fq_quantize_act(Qb)
            s["q"], s["qs"] = qc.view(H, R, GROUP), qs.view(H, R)
            s["k"], s["v"] = fq.fq_kv4_pack(k, False), fq.fq_kv4_pack(v, True)
    elif kind == "cache":
        s["k"], s["v"] = _int4(g, case["H"], case["T"], GROUP), _int4(g, case["H"], case["T"], GROUP)
    else:
        N, K = case["N"], case["K"]
        w = torch.randn((N, K), generator=g, device="cuda") * 0.02
        s["w"] = (w * torch.exp(0.5 * torch.randn((1, K), generator=g, device="cuda"))).to(torch.bfloat16)
    return s


def prepare(case, seed):
    s = _inputs(case, seed, raw=False)
    if case["kind"] == "block":
        # the serving loop's graph: captured once on buffers that stay, replayed for every token
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            _block(s)
            side.synchronize()
            s["graph"] = torch.cuda.CUDAGraph()
            with torch.cuda.graph(s["graph"], stream=side):
                s["out"] = _block(s)
        torch.cuda.current_stream().wait_stream(side)
    return s


# ---- one pass -----------------------------------------------------------------------------------------------

def _quantized(x, N):
    """(codes, scales, workspace, whether the quantiser has prepared it) of a layer's activations."""
    need = fq.fq_w4a8_gemm_workspace_bytes(x.shape[0], N, x.shape[1])
    ws = torch.empty((need,), dtype=torch.uint8, device=x.device) if need else None
    a, scale = fq.fq_quantize_act(x, workspace=ws)
    return a, scale, ws


def _ffn(x, gu, down, res, F):
    """Gate/up with the fused epilogue, its output as FP8 codes, down projection + residual."""
    D = res.shape[1]
    a, scale, ws = _quantized(x, 2 * F)
    need = fq.fq_w4a8_gemm_workspace_bytes(x.shape[0], D, F)
    nws = torch.empty((need,), dtype=torch.uint8, device=x.device) if need else None
    h, hc, hs = fq.fq_w4a8_gemm_swiglu_quant(a, scale, gu[0], gu[1], 1.0, 2 * F, workspace=ws,
                                             workspace_prepared=ws is not None, next_workspace=nws)
    y = fq.fq_w4a8_gemm_add(hc, hs, down[0], down[1], 1.0, D, res, workspace=nws, workspace_prepared=nws is not None)
    return h, hc, hs, y


def _block(s):
    c = s["case"]
    qkv = fq.fq_w4a8_linear(s["x"], s["qkv"][0], s["qkv"][1], 1.0, c["qkv"])
    a, scale, ws = _quantized(s["attn"], c["hidden"])
    r = fq.fq_w4a8_gemm_add(a, scale, s["o"][0], s["o"][1], 1.0, c["hidden"], s["res"], workspace=ws,
                            workspace_prepared=ws is not None)
    h, hc, hs, y = _ffn(r, s["gu"], s["down"], r, c["ffn"])
    return qkv, r, h, hc, hs, y


def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind == "linear":
        return fq.fq_w4a8_linear(s["x"], s["w"][0], s["w"][1], 1.0, c["N"])
    if kind == "residual":
        a, scale, ws = _quantized(s["x"], c["N"])
        return a, scale, fq.fq_w4a8_gemm_add(a, scale, s["w"][0], s["w"][1], 1.0, c["N"], s["res"], workspace=ws,
                                             workspace_prepared=ws is not None)
    if kind == "ffn":
        return _ffn(s["x"], s["gu"], s["down"], s["res"], c["ffn"])
    if kind == "block":
        s["graph"].replay()
        return s["out"]
    if kind == "attention":
        H, R = c["H"], c["R"]
        S = fq.fq_kv4_scores(s["q"], s["qs"], s["k"], s["ks"], SQRT_D)
        pc, ps = fq.fq_quantize_act(s["p"])
        return S, pc, ps, fq.fq_kv4_output(pc.view(H, R, -1), ps.view(H, R), s["v"], s["vs"])
    if kind == "cache":
        return fq.fq_kv4_pack(s["k"], False), fq.fq_kv4_pack(s["v"], True)
    lam = fq.fq_cas_scales(s["w"], 0.02)
    n = int(fq.fq_pts_exponent(s["w"], lam)[0])
    q, gs = fq.fq_quantize_weights(s["w"], lam, n)
    return lam, n, q, gs, fq.fq_pack_weights(q)


# ---- what a pass cannot do without --------------------------------------------------------------------------

def _layer_bytes(N, K):
    return N * K // 2 + N * (K // GROUP)


def work(case):
    kind = case["kind"]
    if kind in ("linear", "residual"):
        M, N, K = case["M"], case["N"], case["K"]
        res = (2 * M * N + M * K + 4 * M) if kind == "residual" else 0      # the residual, and the codes that come out
        return {"bytes": _layer_bytes(N, K) + 2 * M * K + 2 * M * N + res, "flops": 2 * M * N * K}
    if kind == "ffn":
        M, D, F = case["M"], case["hidden"], case["ffn"]
        return {"bytes": _layer_bytes(2 * F, D) + _layer_bytes(D, F) + 6 * M * D + 3 * M * F, "flops": 6 * M * D * F}
    if kind == "block":
        M, D, Q, F = case["M"], case["hidden"], case["qkv"], case["ffn"]
        return {"bytes": _layer_bytes(Q, D) + _layer_bytes(D, D) + _layer_bytes(2 * F, D) + _layer_bytes(D, F)
                + 2 * M * Q + 10 * M * D + 3 * M * F, "flops": 2 * M * D * (Q + D + 3 * F)}
    if kind == "attention":
        H, R, T = case["H"], case["R"], case["T"]
        return {"bytes": 2 * H * T * (GROUP // 2 + 1) + H * R * (3 * GROUP + 5 * T), "flops": 4 * H * R * T * GROUP}
    if kind == "cache":
        return {"bytes": 3 * case["H"] * case["T"] * GROUP, "flops": 0}
    N, K = case["N"], case["K"]
    return {"bytes": 2 * N * K + N * K + N * (K // GROUP) + N * K // 2 + 4 * K, "flops": 0}


def tolerance(case):
    """bf16 results of exact products: one rounding is 1.7e-3 of the result (measured against FP64), and sums in another
    FP32 order move a few per cent of the values by one bf16 step.  Along a chain of layers such a step moves some codes
    of the next layer's FP8 input to their neighbours, and where it is the row's largest value it moves that row's scale
    (measured against FP64: 2.6e-3 after a feed-forward block, 5.1e-3 after the four layers of a decoder block)."""
    kind = case["kind"]
    if kind in ("cache", "offline"):
        return "exact"
    if kind == "ffn":
        return {"rel": 1e-2, "max": 0.2, "differ": 8e-3}
    if kind == "block":
        return {"rel": 2e-2, "max": 0.3, "differ": 8e-3}
    return {"rel": 6e-3, "max": 0.04}


# ---- the same in 64 bits ------------------------------------------------------------------------------------

def _decode(codes):
    return codes.view(torch.float8_e4m3fn).to(torch.float64)


def _quant64(x):
    """(codes as FP64 values, scales) of the per-token quantiser: scale absmax / 448 in FP32, FP32 quotient, E4M3."""
    amax = x.float().abs().amax(dim=1)
    s = torch.where(amax == 0, torch.ones_like(amax), (amax.double() / 448.0).float())
    quot = (x.double() / s.double()[:, None]).float().clamp(-448.0, 448.0)
    return quot.to(torch.float8_e4m3fn).to(torch.float64), s


def _gemm64(a, s, layer, N):
    q, gs = layer
    w = (q.double().view(N, -1, GROUP) * _decode(gs)[:, :, None]).view(N, -1)
    return (a @ w.t()) * s.double()[:, None]


def _ffn64(x, gu, down, res, F):
    a, s = _quant64(x)
    y = _gemm64(a, s, gu, 2 * F)
    gate, up = y[:, 0::2], y[:, 1::2]
    h = gate / (1.0 + torch.exp(-gate)) * up
    hc, hs = _quant64(h.to(torch.bfloat16))
    return h, hs, _gemm64(hc, hs, down, res.shape[1]) + res.double()


def exact(case, seed):
    s, kind = _inputs(case, seed, raw=True), case["kind"]
    if kind == "linear":
        a, sc = _quant64(s["x"])
        return _gemm64(a, sc, s["w"], case["N"])
    if kind == "residual":
        a, sc = _quant64(s["x"])
        return None, sc.double(), _gemm64(a, sc, s["w"], case["N"]) + s["res"].double()
    if kind == "ffn":
        h, hs, y = _ffn64(s["x"], s["gu"], s["down"], s["res"], case["ffn"])
        return h, None, hs.double(), y
    if kind == "block":
        a, sc = _quant64(s["x"])
        qkv = _gemm64(a, sc, s["qkv"], case["qkv"])
        a, sc = _quant64(s["attn"])
        r = _gemm64(a, sc, s["o"], case["hidden"]) + s["res"].double()
        rb = r.to(torch.bfloat16)
        h, hs, y = _ffn64(rb, s["gu"], s["down"], rb, case["ffn"])
        return qkv, r, h, None, hs.double(), y
    if kind == "attention":
        H, R, T = case["H"], case["R"], case["T"]
        q, qs = _quant64(s["q"])
        p, ps = _quant64(s["p"])
        S = torch.empty((H, R, T), dtype=torch.float64, device="cuda")
        O = torch.empty((H, R, GROUP), dtype=torch.float64, device="cuda")
        for h in range(H):
            k = s["k"][h].double() * _decode(s["ks"][h])[:, None]
            v = s["v"][h].double() * _decode(s["vs"][h])[:, None]
            rows = slice(h * R, h * R + R)
            S[h] = (q[rows] @ k.t()) * (qs[rows].double()[:, None] * SQRT_D)
            O[h] = (p[rows, :T] @ v) * ps[rows].double()[:, None]
        return S, None, ps.double(), O
    if kind == "offline":
        mean = s["w"].double().abs().mean(dim=0)
        return torch.where(mean == 0, torch.ones_like(mean), 0.02 / mean), None, None, None, None
    return None
