"""What a call without tiles runs where the model's pick leaves blocks waiting that another arrangement would hold at once, and which
calls of wide n-tiles are split (host only)."""
import random

import pytest

import paper_2506_22169_amd as mcf
from paper_2506_22169_amd.binding import call_tiles, eval_tiles, list_candidates, make_problem


def _feasible(t, p, softmax):
    """Built, within LDS and registers, no spills in loops.  (Not always a candidate of the picker, which also asks that a tile pads little.)"""
    return eval_tiles(p, t.mb, t.rg, t.ns, t.nj, tl=t.tl, softmax=softmax).feasible


def _ran(b, M, K, N, L, causal=False, dtype="bf16", off=None, **kw):
    p = make_problem(b, M, K, N, L, dtype, b_stride=(N * K, 1, K))
    t, ranges = call_tiles(p, True, causal_offset=(N - M if off is None else off) if causal else None, **kw)
    return (t.mb, t.rg, t.ns, t.nj, t.tl), ranges, t, p


@pytest.mark.parametrize("call,run", [
    (dict(b=103, M=1088, K=192, N=512, L=192), (1, 4, 1, 1, 192)),                  # 1751 blocks of 64 rows, one a unit: 95 -> 54 us
    (dict(b=40, M=1216, K=128, N=1280, L=128, dtype="f16"), (1, 8, 1, 2, 128)),      # 760 blocks of 64 rows: 62 -> 39 us
    (dict(b=35, M=1364, K=128, N=1096, L=128, dtype="f16"), (1, 4, 1, 1, 128)),      # less than a tenth to win: the pick
    (dict(b=64, M=4096, K=128, N=4096, L=128), (1, 8, 1, 2, 128)),
    (dict(b=14, M=3072, K=64, N=3072, L=64, causal=True), None),                     # 168 blocks of unequal length: smaller ones
])
def test_arrangement_of_many_blocks(call, run):
    got, ranges, t, p = _ran(**call)
    assert ranges == 1 and t.scratch_bytes == 0
    if run is None:
        q = mcf.pick_tiles(p, True)
        assert t.tm < q.tm and t.blocks > q.blocks
    else:
        assert got == run


def test_what_is_left_alone():
    """Calls of 128 blocks and fewer (n may be split), given tiles, T_L < L; and an arrangement that is taken in their place is feasible and one
    that leaves more than 128 blocks, for any size and offset."""
    rng = random.Random(4)
    moved = 0
    for _ in range(1500):
        K = rng.choice([32, 64, 80, 96, 128, 160, 192, 256])
        b, M, N = rng.randint(1, 200), rng.choice([1, 7, 64, 333, 1000, 4096, rng.randint(1, 5000)]), rng.choice([1, 64, 777, rng.randint(1, 9000)])
        causal = rng.random() < 0.5
        off = rng.choice([0, N - M, -M // 2, N, -M - 5, 10**9, -10**9])
        got, ranges, t, p = _ran(b, M, K, N, K, causal, off=off)
        q = mcf.pick_tiles(p, True)
        if q.blocks <= 128:
            assert (t.mb, t.rg) == (q.mb, q.rg) and t.blocks == q.blocks
        elif t.blocks != q.blocks:
            moved += 1
            assert t.blocks > 128 and ranges == 1 and t.tl == K and t.scratch_bytes == 0 and _feasible(t, p, True)
        given = list_candidates(p, True)[0]
        assert _ran(b, M, K, N, K, causal, off=off, tiles=(given.mb, given.rg, given.ns, given.nj, given.tl))[0][:4] == (given.mb, given.rg, given.ns, given.nj)
    assert moved > 50


def test_what_plain_calls_move_to():
    """The same of plain chains, whose T_L may change with the arrangement."""
    rng = random.Random(5)
    moved = other_tl = 0
    for _ in range(1500):
        K, L = rng.choice([(32, 32), (64, 64), (64, 128), (64, 256), (128, 64), (96, 96), (192, 192), (256, 256)])
        b, M, N = rng.randint(1, 100), rng.choice([64, 333, 1000, rng.randint(1, 4000)]), 8 * rng.randint(1, 400)
        p = make_problem(b, M, K, N, L, rng.choice(["f16", "bf16"]))
        t, ranges = call_tiles(p, False)
        q = mcf.pick_tiles(p, False)
        if q.blocks <= 128:
            assert t.blocks == q.blocks and t.tl == q.tl
        elif t.blocks != q.blocks:
            moved += 1
            other_tl += t.tl != q.tl
            assert t.blocks > 128 and ranges == 1 and t.scratch_bytes == 0 and L % t.tl == 0 and _feasible(t, p, False)
    assert moved > 50 and other_tl > 5


# decode calls of more blocks than compute units; us: the pick's time, the time of what runs
@pytest.mark.parametrize("b,M,K,N,run,us", [(1024, 1, 128, 2048, (1, 2, 2, 1), (189.4, 178.6)), (512, 4, 64, 4096, (1, 2, 2, 1), (97.6, 88.4)),
                                            (512, 1, 96, 4096, (1, 2, 2, 1), (136.2, 136.2)), (1024, 1, 64, 2048, (1, 2, 2, 2), (97.1, 94.4))])
def test_decode_calls_of_many_blocks(b, M, K, N, run, us):
    got, ranges, t, _ = _ran(b, M, K, N, K)
    assert got == run + (K,) and ranges == 1 and t.blocks == b


@pytest.mark.parametrize("call,tm", [
    ((51, 715, 32, 744, 32), 256),                    # 1173 blocks of 32 rows: 15.3 -> 8.2 - 8.8 us
    ((92, 3264, 64, 128, 128), 256),
    ((64, 512, 64, 512, 64), 128),
    ((16, 4096, 32, 1024, 32), 256),
])
def test_arrangement_of_many_plain_blocks(call, tm):
    p = make_problem(*call, "bf16")
    t, ranges = call_tiles(p, False)
    assert ranges == 1 and t.scratch_bytes == 0 and t.blocks > 128 and t.tm == tm


# registers: what lets a compute unit hold two blocks of four waves (256) or of eight (128)
@pytest.mark.parametrize("tiles,softmax,registers", [((1, 4, 1, 4), True, 256), ((2, 4, 1, 2), True, 256), ((2, 2, 2, 2), True, 256),
                                                     ((2, 4, 2, 2), True, 256), ((1, 4, 2, 2), False, 128), ((1, 8, 1, 2), False, 128)])
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_kernels_of_32_keep_their_blocks(tiles, softmax, registers, dtype):
    p = make_problem(96, 512, 32, 512, 32, dtype, b_stride=(512 * 32, 1, 32) if softmax else None)
    t = eval_tiles(p, *tiles, softmax=softmax)
    assert t.vgpr_used <= registers and t.scratch_bytes == 0 and t.stages == 2


@pytest.mark.parametrize("K,L,tiles", [(64, 64, (2, 4, 1, 2)), (64, 64, (2, 2, 2, 2)), (128, 64, (2, 4, 1, 2)), (32, 32, (4, 1, 4, 1)),
                                       (32, 32, (4, 2, 2, 1))])
def test_pipelined_where_the_registers_hold_it(K, L, tiles):
    """Rings of their own for B and D (stages 2), which these ran before more than 320 estimated registers were refused, and without spills."""
    t = eval_tiles(make_problem(32, 2048, K, 2048, L, "f16", b_stride=(2048 * K, 1, K)), *tiles, softmax=True)
    assert t.stages == 2 and t.scratch_bytes == 0


@pytest.mark.parametrize("call,kind,ranges", [
    ((3, 300, 128, 1500, 128), 1, 4),      # twelve n-tiles of 48 KiB
    ((2, 500, 160, 1400, 160), 0, 4),      # eleven of 80 KiB
    ((1, 132, 160, 816, 160), 0, 3),
    ((2, 1241, 192, 616, 192), 0, 1),      # ten of 48 KiB, but 1.9 MB of results a range
    ((20, 192, 64, 2624, 64), 1, 2),       # ten n-tiles saved: whatever the results take
    ((4, 128, 64, 512, 64), 1, 1),
])
def test_ranges_of_wide_n_tiles(call, kind, ranges):
    b, M, K, N, L = call
    assert call_tiles(make_problem(*call, "f16", b_stride=(N * K, 1, K) if kind else None), bool(kind))[1] == ranges
