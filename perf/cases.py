"""Performance cases of the fused chains: the calls a user of this package makes, over the range of
sizes it is used for.

A case is a dict of plain values:
  kind        "chain"   E = (A.B).D                         gemm_chain
              "attn"    E = softmax_rows(scale A.B).D       softmax_gemm_chain
              "causal"  the same under a causal mask        causal_softmax_gemm_chain
              "chain3"  G = (E).F, E a plain chain          gemm_chain3
              "attn3"   G = (E).F, E a softmax chain        gemm_chain3
  batch, M, K, N, L (and P for the chains of three), dtype "f16" | "bf16", out "same" | "f32".
Plain chains hold B as [b,K,N]; attention holds it as the key matrix [b,N,K] and hands over a
transposed view, as it comes out of a projection.  Entries are U(-1,1) for plain chains and N(0,1)
for attention, the softmax scale is 1/sqrt(K), and the mask of a causal case ends in the last row
and column (offset N - M), so M < N is the next piece of a longer sequence.
"""
import math

import torch

import paper_2506_22169_amd as mcf

_DTYPES = {"f16": torch.float16, "bf16": torch.bfloat16}


def _case(kind, batch, M, K, N, L, dtype, P=0, out="same", name=None):
    c = {"kind": kind, "batch": batch, "M": M, "K": K, "N": N, "L": L, "P": P, "dtype": dtype, "out": out}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # one small chain: the latency of a single call (128 KiB in, 128 KiB out)
        _case("chain", 1, 1024, 64, 128, 64, "f16", name="chain_single_small"),
        # the batched chain of the benchmark: attention-shaped, without the softmax
        _case("chain", 64, 512, 64, 512, 64, "f16", name="chain_batched"),
        # a low-rank chain: K = L = 32 over long M, the most memory-bound of the plain chains
        _case("chain", 16, 4096, 32, 1024, 32, "bf16", name="chain_low_rank"),
        # the longest reduction of the paper's table: K beyond what a block holds, one batch
        _case("chain", 1, 512, 1024, 512, 256, "f16", name="chain_long_k"),
        # sizes that divide no tile, a head size that is no power of two, fp32 results for an accumulation outside
        _case("chain", 40, 1000, 96, 776, 96, "bf16", out="f32", name="chain_ragged_f32"),
        # self-attention of an encoder: 8 sequences of 512 tokens, 12 heads of 64
        _case("attn", 96, 512, 64, 512, 64, "f16", name="attn_encoder"),
        # long-sequence self-attention: 4 sequences of 4096 tokens, 16 heads of 128
        _case("attn", 64, 4096, 128, 4096, 128, "bf16", name="attn_long"),
        # prefill of a decoder: 1 sequence of 4096 tokens, 32 heads of 128, causal
        _case("causal", 32, 4096, 128, 4096, 128, "bf16", name="causal_prefill"),
        # the next piece of a prompt against what is cached, ragged, 2 x 20 heads of 80
        _case("causal", 40, 333, 80, 1357, 80, "f16", name="causal_chunk_ragged"),
        # decoding one token against 8192 cached ones, 32 heads of 128
        _case("attn", 32, 1, 128, 8192, 128, "bf16", name="attn_decode"),
        # three plain GEMMs, the benchmark's batched shape
        _case("chain3", 64, 512, 64, 512, 64, "f16", P=64, name="chain3_batched"),
        # attention with its projection behind it: 2 sequences of 2048 tokens, 16 heads of 128
        _case("attn3", 32, 2048, 128, 2048, 128, "bf16", P=128, name="attn3_projection"),
    ]


# (K, L) with the whole K on chip, those of the k loop, and (K, L, P) of the chains of three
_WHOLE_K = [(32, 32), (64, 64), (64, 64), (128, 128), (128, 128), (64, 128), (128, 64), (64, 256), (256, 256), (80, 80), (96, 96), (160, 160),
            (192, 192)]
_HEADS = [64, 64, 128, 128, 80, 96, 160, 192, 256]
_THREE = [(64, 64, 64), (128, 128, 128), (64, 128, 128), (128, 64, 64), (64, 64, 128)]
_MOST_FLOPS, _MOST_BYTES = 2.0e11, 2.0e8


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["chain", "chain", "attn", "attn", "causal", "chain3", "attn3", "long_k", "decode"])
    dtype = rng.choice(["f16", "bf16"])
    out = "f32" if rng.random() < 0.15 else "same"
    P = 0
    M = _log_int(rng, 128, 4096)
    N = _log_int(rng, 128, 4096)
    batch = _log_int(rng, 1, 128)
    if kind == "chain":
        K, L = rng.choice(_WHOLE_K)
    elif kind == "long_k":
        K, L = 128 * rng.randint(3, 8), rng.choice([64, 128, 256])
        M, N, batch = _log_int(rng, 128, 2048), _log_int(rng, 128, 2048), _log_int(rng, 1, 16)
    elif kind in ("chain3", "attn3"):
        K, L, P = rng.choice(_THREE)
    else:
        K = L = rng.choice(_HEADS)
        if kind == "decode":  # one token or a few speculated ones (or query heads that share their keys)
            M, N, batch = rng.choice([1, 1, 2, 4, 5, 8]), _log_int(rng, 512, 16384), _log_int(rng, 4, 256)
        elif kind == "causal":
            N = M if rng.random() < 0.5 else max(N, M)
    # half of the sizes are round, as most users choose them, the others as they come; an N-contiguous B wants multiples of 8
    if rng.random() < 0.5 and M >= 128:
        M = 64 * max(1, round(M / 64))
        N = M if kind == "causal" and N < M else 64 * max(1, round(N / 64))
    if kind in ("chain", "long_k", "chain3"):
        N = 8 * max(1, round(N / 8))
    kind = {"long_k": "chain", "decode": "attn"}.get(kind, kind)
    if kind == "causal":
        N = max(N, M)
    one = _case(kind, 1, M, K, N, L, dtype, P, out)
    w = work(one)
    fits = int(min(_MOST_FLOPS / w["flops"], _MOST_BYTES / w["bytes"]))
    one["batch"] = max(1, min(batch, fits))
    return one


def prepare(case, seed):
    dtype = _DTYPES[case["dtype"]]
    attention = case["kind"] in ("attn", "causal", "attn3")
    b, M, K, N, L, P = (case[k] for k in ("batch", "M", "K", "N", "L", "P"))
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)

    def entries(*shape):
        t = torch.empty(shape, dtype=torch.float32, device="cuda")
        t = t.normal_(generator=gen) if attention else t.uniform_(-1, 1, generator=gen)
        return t.to(dtype)

    s = {"kind": case["kind"], "A": entries(b, M, K), "scale": 1.0 / math.sqrt(K), "offset": N - M, "out": None}
    s["B"] = entries(b, N, K).transpose(1, 2) if attention else entries(b, K, N)
    s["D"] = entries(b, N, L)
    if P:
        s["F"] = entries(b, L, P)
    if case["out"] == "f32":  # fp32 results are asked for by handing over where they go
        s["out"] = torch.empty((b, M, P or L), dtype=torch.float32, device="cuda")
    return s


def run(state):
    kind, A, B, D, out = state["kind"], state["A"], state["B"], state["D"], state["out"]
    if kind == "chain":
        return mcf.gemm_chain(A, B, D, out=out)
    if kind == "attn":
        return mcf.softmax_gemm_chain(A, B, D, state["scale"], out=out)
    if kind == "causal":
        return mcf.causal_softmax_gemm_chain(A, B, D, state["scale"], state["offset"], out=out)
    return mcf.gemm_chain3(A, B, D, state["F"], scale=state["scale"] if kind == "attn3" else None, out=out)


def work(case):
    b, M, K, N, L, P = (case[k] for k in ("batch", "M", "K", "N", "L", "P"))
    out_bytes = 4 if case["out"] == "f32" else 2
    pairs = M * N
    if case["kind"] == "causal":  # row i sees N - M + i + 1 columns
        pairs = M * (N - M) + M * (M + 1) // 2
    return {"bytes": b * (2 * (M * K + K * N + N * L + L * P) + out_bytes * M * (P or L)),
            "flops": 2 * b * (pairs * (K + L) + M * L * P)}


def tolerance(case):
    """Four times the distance measured between these kernels and the same chain in 64 bits (norm / largest): 2.95e-4 /
    1.3e-3 in fp16 and 2.4e-3 / 1.2e-2 in bf16 from the rounding of the intermediate and of the result, 3.6e-4 / 1.7e-3
    and 2.9e-3 / 1.5e-2 for the chains of three with one rounding more, and 2.4e-2 at the most for the first rows of a
    causal mask in bf16, which average a few columns only and are larger than the rest."""
    three = case["P"] > 0
    if case["dtype"] == "f16":
        return {"rel": 1.5e-3 if three else 1.2e-3, "max": 1.2e-2 if case["kind"] == "causal" else 7.0e-3}
    return {"rel": 1.2e-2 if three else 1.0e-2, "max": 1.0e-1 if case["kind"] == "causal" else 6.0e-2}
