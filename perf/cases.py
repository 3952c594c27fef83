"""The work that is timed for this framework: its products and decode attention, called as a serving program calls them.

Sizes are those of an 8B-class decoder (hidden 4096, FFN 14336, fused QKV 6144, 32 query heads of 128, 8 or 32 key/value
heads), of mixture-of-experts layers (32 or 6 experts on a GPU) and of latent attention (576-wide rows, 16 or 128 heads),
with square and odd products beside them.  A program keeps the probed topology, its weights and its output buffers; the
activations and caches are drawn by a seeded generator on the GPU, N(0, 1), the weights N(0, 0.02).
"""
import functools
import math

import torch

import paper_2609_24270_amd as asym

DEV = "cuda:0"


def _gemm(M, N, K, layout="nk"):
    return {"op": "gemm", "M": M, "N": N, "K": K, "layout": layout}


def _grouped(G, M, N, K):
    return {"op": "grouped", "G": G, "M": M, "N": N, "K": K}


def _attn(B, Hkv, S, paged):
    return {"op": "attn", "B": B, "Hq": 32, "Hkv": Hkv, "S": S, "paged": paged}


def _mla(B, Hq, S):
    return {"op": "mla", "B": B, "Hq": Hq, "S": S}


def listed():
    return [
        # the smallest call: a small square product, where launches and latency count
        dict(_gemm(512, 512, 512), name="gemm_512"),
        # one decode step of 32 requests through the FFN's up projection: the weights are read once
        dict(_gemm(32, 14336, 4096), name="gemm_decode_up"),
        # a 512-token prefill chunk through the fused QKV projection
        dict(_gemm(512, 6144, 4096), name="gemm_chunk_qkv"),
        # a 4096-token prefill through the FFN's up projection
        dict(_gemm(4096, 14336, 4096), name="gemm_prefill_up"),
        # the headline square product
        dict(_gemm(8192, 8192, 8192), name="gemm_8192"),
        # sizes that are a multiple of nothing: rows of odd length start on 2-byte boundaries
        dict(_gemm(1000, 3001, 1501), name="gemm_odd"),
        # weights that lie [K][N], as a program that multiplies x @ W stores them
        dict(_gemm(2048, 6144, 4096, "kn"), name="gemm_kn"),
        # an expert layer during prefill: 32 experts with about 192 tokens each
        dict(_grouped(32, 192, 4096, 4096), name="experts_prefill"),
        # an expert layer during decode: about 20 tokens each
        dict(_grouped(32, 20, 4096, 2048), name="experts_decode"),
        # one decode step of 16 requests over dense 8000-token caches, grouped-query heads
        dict(_attn(16, 8, 8000, False), name="attn_gqa"),
        # a small batch over paged caches, pages wherever the allocator put them
        dict(_attn(4, 8, 4000, True), name="attn_paged"),
        # latent-attention decode with all 128 heads on one GPU
        dict(_mla(16, 128, 8192), name="mla_128"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(("gemm", "gemm", "gemm", "grouped", "attn", "mla"))
    if op == "gemm":
        while True:
            M, N, K = _log(rng, 1, 8192), _log(rng, 128, 16384), _log(rng, 128, 16384)
            if rng.random() < 0.85:  # rows of 16 bytes and more are the rule; any length is taken
                N, K = (N + 7) // 8 * 8, (K + 7) // 8 * 8
            if M * N * K <= 8192 ** 3:
                return _gemm(M, N, K, "kn" if rng.random() < 0.15 else "nk")
    if op == "grouped":
        G = rng.choice((6, 8, 16, 32))
        M = _log(rng, 8, 6144 // G)
        N, K = rng.choice(((6144, 7168), (7168, 3072), (4096, 4096), (4096, 2048), (2048, 1408), (1000, 2040)))
        return _grouped(G, M, N, K)
    if op == "attn":
        Hkv = rng.choice((8, 8, 32))
        B = _log(rng, 1, 64)
        S = _log(rng, 64, min(32768, (1 << 31) // (512 * B * Hkv)))
        return _attn(B, Hkv, S, rng.random() < 0.5)
    Hq = rng.choice((16, 128))
    B = _log(rng, 1, 64)
    return _mla(B, Hq, _log(rng, 64, min(32768, (1 << 20) // B)))


@functools.lru_cache(maxsize=1)
def _topology():
    return asym.probe_topology(0, asym.PROBE_IDENTITY)


def _rows(case):
    """The experts' row counts: M times a uniform draw from [0.7, 1.3), the same for every seed (a captured
    layer's shape), so that a case's work is one number."""
    g = torch.Generator(device="cpu").manual_seed(5)
    u = torch.rand(case["G"], generator=g, dtype=torch.float64) * 0.6 + 0.7
    return [int(case["M"] * float(x)) for x in u]


def _inputs(case, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)

    def normal(shape, sigma=1.0):
        return (torch.randn(shape, generator=g, device=DEV) * sigma).to(torch.bfloat16)

    op = case["op"]
    if op == "gemm":
        M, N, K = case["M"], case["N"], case["K"]
        return {"A": normal((M, K)), "B": normal((N, K) if case["layout"] == "nk" else (K, N), 0.02)}
    if op == "grouped":
        rows = _rows(case)
        B = torch.empty((case["G"], case["N"], case["K"]), dtype=torch.bfloat16, device=DEV)
        for i in range(case["G"]):
            B[i] = normal((case["N"], case["K"]), 0.02)
        return {"rows": rows, "A": normal((sum(rows), case["K"])), "B": B}
    if op == "attn":
        B, S, Hkv = case["B"], case["S"], case["Hkv"]
        q = normal((B, case["Hq"], 128))
        if not case["paged"]:
            return {"q": q, "k": normal((B, Hkv, S, 128)), "v": normal((B, Hkv, S, 128))}
        pages = (S + asym.PAGE_TOKENS - 1) // asym.PAGE_TOKENS
        n = B * Hkv * pages
        tables = [torch.randperm(n, generator=g, device=DEV).to(torch.int32).view(B, Hkv, pages) for _ in range(2)]
        pools = [normal((n, asym.PAGE_TOKENS, 128)) for _ in range(2)]
        return {"q": q, "k": pools[0], "v": pools[1], "k_pages": tables[0], "v_pages": tables[1]}
    return {"q": normal((case["B"], case["Hq"], 576)), "kv": normal((case["B"], case["S"], 576))}


def prepare(case, seed):
    s = dict(_inputs(case, seed), case=case, topo=_topology())
    if case["op"] == "gemm":
        s["C"] = torch.empty((case["M"], case["N"]), dtype=torch.bfloat16, device=DEV)
    elif case["op"] == "grouped":
        s["C"] = torch.empty((sum(s["rows"]), case["N"]), dtype=torch.bfloat16, device=DEV)
    else:
        d = 128 if case["op"] == "attn" else 512
        s["o"] = torch.empty((case["B"], case["Hq"], d), dtype=torch.bfloat16, device=DEV)
        s["lse"] = torch.empty((case["B"], case["Hq"]), dtype=torch.float32, device=DEV)
    return s


def run(s):
    case = s["case"]
    if case["op"] == "gemm":
        return asym.gemm(s["A"], s["B"], s["C"], topo=s["topo"], b_layout=case["layout"])
    if case["op"] == "grouped":
        return asym.gemm_grouped(s["A"], s["B"], s["rows"], s["C"], topo=s["topo"])
    if case["op"] == "mla":
        asym.mla_decode(s["q"], s["kv"], s["o"], s["lse"], topo=s["topo"])
    elif case["paged"]:
        asym.attn_decode_paged(s["q"], s["k"], s["v"], s["k_pages"], s["v_pages"], case["S"], s["o"], s["lse"],
                               topo=s["topo"])
    else:
        asym.attn_decode(s["q"], s["k"], s["v"], s["o"], s["lse"], topo=s["topo"])
    return {"o": s["o"], "lse": s["lse"]}


def work(case):
    if case["op"] == "gemm":
        M, N, K = case["M"], case["N"], case["K"]
        return {"bytes": 2 * (M * K + N * K + M * N), "flops": 2 * M * N * K}
    if case["op"] == "grouped":
        rows, G, N, K = sum(_rows(case)), case["G"], case["N"], case["K"]
        return {"bytes": 2 * (rows * (K + N) + G * N * K), "flops": 2 * rows * N * K}
    B, Hq, S = case["B"], case["Hq"], case["S"]
    if case["op"] == "attn":
        tables = 8 * B * case["Hkv"] * ((S + asym.PAGE_TOKENS - 1) // asym.PAGE_TOKENS) if case["paged"] else 0
        return {"bytes": 4 * B * case["Hkv"] * S * 128 + 4 * B * Hq * 128 + 4 * B * Hq + tables,
                "flops": 4 * B * Hq * S * 128}
    return {"bytes": 2 * B * S * 576 + 2 * B * Hq * (576 + 512) + 4 * B * Hq, "flops": 2 * B * Hq * S * (576 + 512)}


def tolerance(case):
    # Against 64-bit results, rounded to bf16 or not: products and attention are off by one bf16 rounding (2-norm
    # 1.7e-3, largest 3.9e-3); in attention the probabilities are rounded to bf16 as well, before the sum over tokens.
    return {"rel": 7e-3, "max": 1.6e-2}


def exact(case, seed):
    x = _inputs(case, seed)
    f = torch.float64
    if case["op"] == "gemm":
        B = x["B"].to(f)
        return x["A"].to(f) @ (B.t() if case["layout"] == "nk" else B)
    if case["op"] == "grouped":
        parts = x["A"].to(f).split(x["rows"])
        return torch.cat([a @ x["B"][i].to(f).t() for i, a in enumerate(parts)])
    B, Hq, S = case["B"], case["Hq"], case["S"]
    d = 128 if case["op"] == "attn" else 512
    o = torch.empty((B, Hq, d), dtype=f, device=DEV)
    lse = torch.empty((B, Hq), dtype=f, device=DEV)
    for b in range(B):
        if case["op"] == "mla":
            heads = [(slice(0, Hq), x["kv"][b].to(f), x["kv"][b, :, :512].to(f), 1.0 / math.sqrt(192.0))]
        else:
            heads, G = [], Hq // case["Hkv"]
            for h in range(case["Hkv"]):
                k, v = (x[n][b, h] if not case["paged"] else x[n][x[n + "_pages"][b, h].long()].reshape(-1, 128)[:S]
                        for n in ("k", "v"))
                heads.append((slice(h * G, (h + 1) * G), k.to(f), v.to(f), 1.0 / math.sqrt(128.0)))
        for hs, k, v, scale in heads:
            s = x["q"][b, hs].to(f) @ k.t() * scale
            lse[b, hs] = torch.logsumexp(s, 1)
            o[b, hs] = torch.softmax(s, 1) @ v
    return {"o": o, "lse": lse}
