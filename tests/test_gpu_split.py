"""Chains whose n range is split over blocks (mcf_call with n_split > 1: partial results in a workspace,
put together by a second kernel) against the fp64 oracle: ragged last ranges, more ranges than
n-tiles, ranges a causal mask hides, every way a partial result leaves a block.  Needs an MI355X."""
import numpy as np
import pytest
import torch

import mcf_inputs as mi
import oracle
import paper_2506_22169_amd as mcf
from paper_2506_22169_amd import binding

from gpu_util import TOL, device_inputs, to_device, to_host64

pytestmark = pytest.mark.gpu

# kind, batch, M, K, N, L, P, dtype, offset, tiles (mb, rg, ns, nj[, tl]), ranges
CASES = [
    ("plain", 2, 100, 64, 264, 64, 0, "f16", 0, (1, 1, 4, 1), 2),          # last range: one column group of 8
    ("plain", 3, 333, 32, 1000, 32, 0, "bf16", 0, (1, 8, 1, 2), 99),       # as many ranges as n-tiles
    ("plain", 1, 70, 64, 520, 256, 0, "f16", 0, (1, 2, 2, 1, 64), 3),      # h tiles
    ("plain", 2, 65, 384, 328, 128, 0, "bf16", 0, (1, 1, 8, 1), 2),        # fewer blocks of E than waves
    ("plain", 1, 40, 640, 328, 256, 0, "f16", 0, (1, 1, 4, 1), 3),
    ("softmax", 2, 1, 128, 1061, 128, 0, "bf16", 0, (1, 1, 4, 1), 5),      # one row
    ("softmax", 2, 77, 128, 517, 128, 0, "f16", 0, (1, 2, 2, 1, 64), 4),   # h tiles: the row sums are stored once
    ("softmax", 3, 300, 80, 331, 80, 0, "bf16", 0, (1, 4, 1, 1), 4),       # partial column block, one wave across n
    ("softmax", 1, 129, 192, 300, 192, 0, "f16", 0, (1, 2, 2, 1), 2),
    ("softmax", 2, 130, 64, 400, 64, 0, "bf16", 0, (2, 2, 4, 1), 3),       # two row sets a wave
    ("causal", 2, 333, 64, 461, 64, 0, "f16", 0, (1, 2, 2, 1), 8),         # ranges that early rows do not see
    ("causal", 2, 200, 128, 461, 128, 0, "bf16", -70, (1, 1, 4, 1, 64), 3),  # rows that see nothing
    ("causal", 9, 1100, 64, 700, 64, 0, "f16", -300, (1, 1, 4, 1), 2),     # longest blocks first as well
    ("chain3", 2, 150, 64, 392, 64, 64, "f16", 0, (1, 2, 2, 1), 3),        # the product's partial sums combined first
    ("chain3", 2, 150, 128, 392, 64, 64, "bf16", 0, (1, 4, 1, 1), 2),
    ("attn3", 2, 150, 128, 301, 128, 128, "bf16", 0, (1, 1, 4, 1), 3),
    ("attn3", 1, 150, 64, 301, 64, 128, "f16", 0, (1, 4, 1, 2), 4),
]


def _run(case, out_dtype=None, stream=None):
    kind, b, M, K, N, L, P, dtype, off, tiles, ranges = case
    softmax = kind in ("softmax", "causal", "attn3")
    w = mi.make_problem(b, M, K, N, L, dtype, softmax, "normal" if softmax else "uniform", seed=9100 + M + N)
    x = mi.make_inputs(w)
    A, B, D = device_inputs(w, x)
    F = ref = None
    if kind == "causal":
        ref = oracle.chain_causal(x["A"], x["B"], x["D"], scale=w.scale, causal_offset=off)
    elif P:
        f = mi.to_bits(mi.draw(9100, 4, (b, L, P), w.dist), dtype)
        F = to_device(f, dtype)
        ref = oracle.chain3(x["A"], x["B"], x["D"], mi.from_bits(f, dtype), softmax=softmax, scale=w.scale)
    else:
        ref = oracle.chain(x["A"], x["B"], x["D"], softmax=softmax, scale=w.scale)
    code = {"plain": 0, "chain3": 0, "softmax": 1, "attn3": 1, "causal": 2}[kind]

    def call(n_split, out=None):
        if out is None and out_dtype is not None:
            out = torch.full((b, M, P or L), 7.0, dtype=out_dtype, device="cuda")
        return binding._call(code, w.scale, off, A, B, D, F, out, tiles, stream, n_split)
    return call, ref, (np.arange(M) + off < 0 if kind == "causal" else np.zeros(M, bool))


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"{c[0]}_{c[1]}x{c[2]}x{c[3]}x{c[4]}x{c[5]}_{c[10]}")
def test_split_ranges_match_the_oracle(case):
    print("case split", case, flush=True)
    call, ref, blind = _run(case)
    got = to_host64(call(case[10]), case[7])
    assert np.isfinite(got).all()
    err, scale = np.max(np.abs(got - ref)), np.max(np.abs(ref))
    assert err <= TOL * scale, f"{case}: {err:.4g} > {TOL} * {scale:.4g}"
    assert not got[:, blind].any()
    # fp32 results: the same sums, not rounded
    call32, _, _ = _run(case, out_dtype=torch.float32)
    e32 = call32(case[10])
    torch.cuda.synchronize()
    assert torch.equal(e32.to(torch.float16 if case[7] == "f16" else torch.bfloat16), call(case[10]))


def test_split_ranges_on_streams_and_in_graphs():
    """Three streams at once, each call with a workspace of its own, and replays of a captured call: bit
    for bit what one call alone gives."""
    case = ("softmax", 4, 64, 64, 1000, 64, 0, "f16", 0, (1, 1, 4, 1), 4)
    call, _, _ = _run(case)
    alone = call(4)
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(3)]
    runs = [_run(case, stream=s)[0] for s in streams]
    outs = [torch.empty_like(alone) for _ in streams]
    torch.cuda.synchronize()
    print("case split streams", flush=True)
    for _ in range(20):
        for run, out in zip(runs, outs):
            run(4, out)
    torch.cuda.synchronize()
    assert all(torch.equal(o, alone) for o in outs)
    E = torch.zeros_like(alone)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        call(4, E)
    for rep in range(4):
        print(f"case split graph replay {rep}", flush=True)
        E.fill_(-3.0)
        call(4)                      # eager work between the replays
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(E, alone)


# kind, batch, M, K, N, L, dtype: calls that the library splits, and calls whose waves it arranges behind the model's pick
CHOSEN = [("softmax", 8, 1, 128, 2500, 128, "bf16"), ("softmax", 2, 70, 64, 3001, 64, "f16"), ("plain", 1, 300, 512, 1000, 128, "f16"),
          ("plain", 2, 129, 64, 2056, 256, "bf16"), ("plain", 15, 610, 64, 736, 128, "bf16"), ("plain", 6, 1635, 64, 800, 128, "bf16"),
          ("softmax", 6, 1718, 64, 735, 128, "f16"), ("softmax", 12, 687, 80, 66, 80, "bf16")]


@pytest.mark.parametrize("case", CHOSEN, ids=str)
def test_calls_without_tiles_match_the_oracle(case):
    """The path a program takes: neither tiles nor ranges given."""
    kind, b, M, K, N, L, dtype = case
    softmax = kind == "softmax"
    w = mi.make_problem(b, M, K, N, L, dtype, softmax, "normal" if softmax else "uniform", seed=9170 + N)
    x = mi.make_inputs(w)
    A, B, D = device_inputs(w, x)
    problem = binding.make_problem(b, M, K, N, L, dtype, b_stride=(N * K, 1, K) if softmax else None)
    t, ranges = mcf.call_tiles(problem, softmax)
    q = mcf.pick_tiles(problem, softmax)
    assert ranges > 1 or (t.ns, t.nj) != (q.ns, q.nj)
    print("case chosen", case, (t.mb, t.rg, t.ns, t.nj, t.tl), ranges, flush=True)
    for out_dtype in (None, torch.float32):
        out = None if out_dtype is None else torch.empty((b, M, L), dtype=out_dtype, device="cuda")
        E = mcf.softmax_gemm_chain(A, B, D, w.scale, out=out) if softmax else mcf.gemm_chain(A, B, D, out=out)
        got = E.double().cpu().numpy() if out_dtype else to_host64(E, dtype)
        ref = oracle.chain(x["A"], x["B"], x["D"], softmax=softmax, scale=w.scale)
        assert np.max(np.abs(got - ref)) <= TOL * np.max(np.abs(ref))


# calls of more than 128 blocks that run another arrangement, one with another T_L, than the model's pick
MOVED = [("plain", 22, 765, 64, 152, 256, "bf16"), ("plain", 8, 897, 64, 384, 256, "f16"), ("softmax", 37, 409, 96, 124, 96, "bf16"),
         ("softmax", 133, 80, 64, 363, 64, "f16"), ("softmax", 300, 4, 64, 1096, 64, "bf16"), ("causal", 43, 352, 96, 252, 96, "bf16"),
         ("causal", 96, 283, 192, 122, 192, "f16")]


@pytest.mark.parametrize("case", MOVED, ids=str)
def test_calls_of_many_blocks_match_the_oracle(case):
    kind, b, M, K, N, L, dtype = case
    softmax, off = kind != "plain", N - M
    w = mi.make_problem(b, M, K, N, L, dtype, softmax, "normal" if softmax else "uniform", seed=9180 + N)
    x = mi.make_inputs(w)
    A, B, D = device_inputs(w, x)
    problem = binding.make_problem(b, M, K, N, L, dtype, b_stride=(N * K, 1, K) if softmax else None)
    t, ranges = mcf.call_tiles(problem, softmax, causal_offset=off if kind == "causal" else None)
    q = mcf.pick_tiles(problem, softmax)
    assert ranges == 1 and (t.mb, t.rg, t.ns, t.nj, t.tl) != (q.mb, q.rg, q.ns, q.nj, q.tl)
    print("case moved", case, (t.mb, t.rg, t.ns, t.nj, t.tl), flush=True)
    if kind == "causal":
        E, ref = mcf.causal_softmax_gemm_chain(A, B, D, w.scale, off), oracle.chain_causal(x["A"], x["B"], x["D"], scale=w.scale, causal_offset=off)
    else:
        E = mcf.softmax_gemm_chain(A, B, D, w.scale) if softmax else mcf.gemm_chain(A, B, D)
        ref = oracle.chain(x["A"], x["B"], x["D"], softmax=softmax, scale=w.scale)
    assert np.max(np.abs(to_host64(E, dtype) - ref)) <= TOL * np.max(np.abs(ref))


@pytest.mark.parametrize("b,M,K,N,off", [(32, 1, 128, 8192, 5000), (3, 70, 64, 6000, 4000), (2, 33, 96, 4097, 4096 - 32), (9, 200, 64, 5000, 2049)])
def test_ranges_end_with_what_a_mask_leaves(b, M, K, N, off):
    """Ranges that the library chooses under a mask stop at the columns the last row sees."""
    w = mi.make_problem(b, M, K, N, K, "f16", True, "normal", seed=9150 + off)
    x = mi.make_inputs(w)
    A, B, D = device_inputs(w, x)
    assert mcf.call_tiles(binding.make_problem(b, M, K, N, K, "f16", b_stride=(N * K, 1, K)), True, causal_offset=off)[1] > 1
    print("case masked ranges", b, M, K, N, off, flush=True)
    got = to_host64(mcf.causal_softmax_gemm_chain(A, B, D, w.scale, off), "f16")
    ref = oracle.chain_causal(x["A"], x["B"], x["D"], scale=w.scale, causal_offset=off)
    assert np.max(np.abs(got - ref)) <= TOL * np.max(np.abs(ref))


@pytest.mark.skipif(torch.cuda.device_count() < 2, reason="needs a second device")
def test_workspace_lives_with_the_operands():
    """Operands and stream of a device that is not the current one: so does the workspace."""
    case = ("softmax", 4, 64, 64, 1000, 64, 0, "f16", 0, (1, 1, 4, 1), 4)
    call, _, _ = _run(case)
    alone = call(4)
    with torch.cuda.device(1):
        there, _, _ = _run(case, stream=torch.cuda.Stream())
        torch.cuda.synchronize()
        before = torch.cuda.memory_stats(0)["allocation.all.allocated"]
    print("case split on the second device", flush=True)
    E = there(4)
    torch.cuda.synchronize(1)
    assert E.device.index == 1 and torch.equal(E.cpu(), alone.cpu())
    assert torch.cuda.memory_stats(0)["allocation.all.allocated"] == before
