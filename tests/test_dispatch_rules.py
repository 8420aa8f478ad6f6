"""What a call without an arrangement runs, on the host: which calls split n, into how much, and
that a split call asks for the workspace its ranges need."""
import ctypes
import random

import pytest

import paper_2506_22169_amd as mcf
from paper_2506_22169_amd import binding
from paper_2506_22169_amd.binding import make_problem


def _workspace(batch, M, K, N, L, dtype="f16", kind=0, P=0, out_f32=False, n_split=0, tiles=None):
    lib = binding.load_library()
    c = binding.Call()
    c.problem = make_problem(batch, M, K, N, L, dtype, b_stride=(N * K, 1, K) if kind else None)
    if out_f32:
        c.problem.out_dtype = binding.MCF_F32
    c.P, c.softmax, c.causal, c.scale, c.n_split, c.causal_offset = P, int(kind > 0), int(kind == 2), 1.0, n_split, N - M
    base = 1 << 40  # addresses are compared, never read
    c.A, c.B, c.D, c.E, c.F = base, base << 1, base << 2, base << 3, base << 4 if P else None
    if tiles is not None:
        t = binding.Tiles(mb=tiles[0], rg=tiles[1], ns=tiles[2], nj=tiles[3])
        c.tiles = ctypes.addressof(t)
    need = ctypes.c_int64(-1)
    status = lib.mcf_call_workspace(ctypes.byref(c), ctypes.byref(need))
    assert status == 0, status
    rows = batch * M * ((P or L) + (4 if kind else 0)) * 4
    assert need.value % rows == 0
    return need.value // rows  # ranges; 0: n is not split


@pytest.mark.parametrize("out_f32", [False, True])
def test_calls_that_split(out_f32):
    assert _workspace(32, 1, 128, 8192, 128, "bf16", 1, out_f32=out_f32) >= 4       # one token against a long cache
    assert _workspace(1, 639, 1024, 664, 128, out_f32=out_f32) >= 8                  # a k loop on ten blocks
    assert _workspace(1, 512, 1024, 512, 256, out_f32=out_f32) == 2                  # nine items of a k loop fewer
    assert _workspace(1, 209, 96, 3003, 96, "f16", 2, out_f32=out_f32) >= 2


def test_calls_that_do_not_split():
    assert _workspace(64, 512, 64, 512, 64) == 0            # a block for every compute unit
    assert _workspace(1, 1024, 64, 128, 64) == 0            # one n-tile
    assert _workspace(4, 128, 64, 512, 64, "f16", 1) == 0   # nothing to win: a few n-tiles
    assert _workspace(32, 1, 128, 8192, 128, "bf16", 1, n_split=1) == 0
    assert _workspace(5, 953, 64, 3696, 64, "f16", 0, P=128) == 0  # three GEMMs: a range would round its part of E
    assert _workspace(5, 953, 64, 3696, 64, "f16", 0, P=128, n_split=3) == 3
    assert _workspace(32, 1, 128, 8192, 128, "bf16", 1, tiles=(1, 1, 4, 1)) == 0  # arrangement given
    assert _workspace(32, 1, 128, 8192, 128, "bf16", 1, tiles=(1, 1, 4, 1), n_split=4) == 4


@pytest.mark.parametrize("N", [1, 7, 8, 127, 128, 129, 1000, 1279, 1280, 1288, 4096, 65537, 1 << 20])
@pytest.mark.parametrize("blocks", [1, 3, 85, 127, 128, 129, 256])
def test_ranges_fill_and_do_not_overfill(N, blocks):
    """At most one block a compute unit, and no range without a column, for any N."""
    r = _workspace(blocks, 1, 96, N, 96, "bf16", 1)
    t = mcf.pick_tiles(make_problem(blocks, 1, 96, N, 96, "bf16", b_stride=(N * 96, 1, 96)), True)
    assert r == 0 or (r >= 2 and r * blocks <= 256)
    n_tiles = -(-N // 32)
    assert r <= n_tiles
    assert (r == 0) if 2 * blocks > 256 or N <= 10 * 32 else True
    assert t.blocks == blocks


def _ran(batch, M, K, N, L, kind=0, P=0, dtype="f16", **kw):
    p = make_problem(batch, M, K, N, L, dtype, b_stride=(N * K, 1, K) if kind else None)
    t, ranges = mcf.call_tiles(p, kind > 0, P=P, causal_offset=N - M if kind == 2 else None, **kw)
    return (t.mb, t.rg, t.ns, t.nj, t.tl), ranges, t


def test_calls_say_what_they_run():
    """mcf_call_tiles: the settled arrangement and the ranges, where they differ from the model's pick."""
    # (the arrangement run, the pick): a ragged N that pads least with 32 columns, on eight waves
    for shape, run, picked in (((15, 1635, 64, 4048, 128), (1, 4, 2, 2, 128), (1, 4, 1, 1)),
                               ((128, 2881, 128, 976, 128), (1, 4, 2, 2, 128), (1, 4, 1, 1)),   # ... also with many blocks
                               ((45, 2090, 80, 1248, 80), (1, 4, 2, 2, 80), (1, 4, 1, 1)),
                               ((64, 512, 64, 512, 64), (1, 4, 2, 2, 64), (1, 4, 2, 2))):
        got, ranges, t = _ran(*shape)
        q = mcf.pick_tiles(make_problem(*shape, "f16"))
        assert (got, ranges, (q.mb, q.rg, q.ns, q.nj)) == (run, 1, picked), shape
        assert t.blocks == q.blocks and t.tm == q.tm and t.lds_bytes <= 160 * 1024
    assert _ran(5, 3887, 64, 2207, 64, kind=1)[:2] == ((1, 4, 2, 2, 64), 1)
    assert _ran(35, 1364, 128, 1096, 128, kind=1)[0][:4] == (1, 4, 1, 1)      # softmax, more blocks than compute units: stays
    assert _ran(40, 333, 80, 1357, 80, kind=2)[:2] == ((1, 2, 2, 1, 80), 1)  # rows padded to the pitch: one slice a wave
    assert _ran(32, 1, 128, 8192, 128, kind=1)[1] == 4
    assert _ran(1, 512, 1024, 512, 256)[1] == 2
    # given tiles and ranges are what runs; the calls without a workspace never split
    assert _ran(32, 1, 128, 8192, 128, kind=1, tiles=(1, 1, 4, 1))[:2] == ((1, 1, 4, 1, 128), 1)
    assert _ran(32, 1, 128, 8192, 128, kind=1, tiles=(1, 1, 4, 1, 64), n_split=3)[:2] == ((1, 1, 4, 1, 64), 3)
    assert _ran(32, 1, 128, 8192, 128, kind=1, n_split=1)[1] == 1
    assert _ran(0, 512, 64, 512, 64)[:2] == ((0, 0, 0, 0, 0), 0)             # nothing to compute


def test_call_tiles_of_three_gemms_describe_that_kernel():
    got, ranges, t = _ran(32, 2048, 128, 2048, 128, kind=1, P=128, dtype="bf16")
    assert got == (1, 8, 1, 2, 128) and ranges == 1
    q = mcf.pick_tiles3(make_problem(32, 2048, 128, 2048, 128, "bf16", b_stride=(2048 * 128, 1, 128)), 128, True)
    assert (t.lds_bytes, t.blocks) == (q.lds_bytes, q.blocks)
    with pytest.raises(mcf.McfError):
        _ran(32, 512, 128, 512, 128, P=64)                                   # not built


@pytest.mark.parametrize("kind", [0, 1])
@pytest.mark.parametrize("M,N", [(827, 1112), (128, 4096), (1635, 4048), (64, 64)])
def test_three_gemms_run_the_pick(kind, M, N):
    """No wave or range gets a part of E to round that the model's pick does not give it."""
    for K, L, P in ((64, 64, 64), (128, 64, 64), (64, 64, 128), (128, 128, 128)):
        q = mcf.pick_tiles3(make_problem(3, M, K, N, L, "f16", b_stride=(N * K, 1, K) if kind else None), P, kind > 0)
        assert _ran(3, M, K, N, L, kind=kind, P=P)[:2] == ((q.mb, q.rg, q.ns, q.nj, L), 1)


def test_call_tiles_refuses_what_the_call_refuses():
    lib, t, r = binding.load_library(), binding.Tiles(), ctypes.c_int32(7)
    c = binding.Call()
    assert lib.mcf_call_tiles(None, ctypes.byref(t), ctypes.byref(r)) == 1
    assert lib.mcf_call_tiles(ctypes.byref(c), None, ctypes.byref(r)) == 1
    assert lib.mcf_call_tiles(ctypes.byref(c), ctypes.byref(t), None) == 1
    c.problem, c.scale = make_problem(2, 64, 64, 64, 64, "f16"), 1.0
    c.A, c.B, c.D, c.E = 1 << 40, 1 << 41, 1 << 42, 1 << 40                  # E aliases A
    assert lib.mcf_call_tiles(ctypes.byref(c), ctypes.byref(t), ctypes.byref(r)) == 1
    assert r.value == 0 and t.mb == 0


# Kernels that stand at the edge of a block more or less per compute unit: K, L, P, softmax, B as [b,N,K], arrangement, blocks
RESIDENT = [(32, 32, 0, 1, 0, (1, 4, 1, 1), 5), (32, 32, 0, 1, 1, (1, 2, 2, 1), 5), (64, 64, 0, 0, 0, (1, 4, 2, 2), 2),
            (64, 128, 0, 0, 0, (1, 8, 1, 1), 2), (64, 128, 0, 0, 1, (1, 8, 1, 1), 2), (64, 64, 64, 0, 0, (1, 4, 2, 2), 2),
            (64, 64, 0, 1, 1, (1, 4, 2, 1), 2), (64, 64, 0, 1, 1, (1, 8, 1, 1), 2)]


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("kernel", RESIDENT, ids=str)
def test_blocks_a_compute_unit_holds(kernel, dtype):
    """Registers (allocated by eight, 512 a lane and SIMD) and LDS (160 KiB) leave room for that many blocks,
    and nothing spills in a loop."""
    K, L, P, softmax, nk, tiles, blocks = kernel
    p = make_problem(64, 512, K, 512, L, dtype, b_stride=(512 * K, 1, K) if nk else None)
    t, _ = mcf.call_tiles(p, bool(softmax), P=P, tiles=tiles)
    waves = 512 // ((t.vgpr_used + 7) // 8 * 8)
    assert min(4 * waves // t.waves, 160 * 1024 // t.lds_bytes) >= blocks and t.scratch_bytes == 0


def test_longest_first_only_where_blocks_differ():
    """The order of a masked call's blocks (an internal rule): longest first where the longest is at least an eighth longer
    than the mean, counted here block by block."""
    rule = binding.load_library()._ZN3mcf13longest_firstEllll
    rule.restype, rule.argtypes = ctypes.c_bool, [ctypes.c_int64] * 4
    rng = random.Random(3)
    seen = [0, 0]
    for _ in range(4000):
        M, N, tm = rng.randint(1, rng.choice([40, 4000])), rng.randint(1, rng.choice([40, 9000])), rng.choice([32, 64, 128, 256])
        off = rng.choice([0, N - M, N, N - 1, -M // 2, N // 2, rng.randint(-M, N)])
        columns = [min(max(tm * (m + 1) + off, 0), N) for m in range(-(-M // tm))]
        longest = min(max(M + off, 0), N)
        want = sum(columns) > 0 and 8 * longest * len(columns) >= 9 * sum(columns)
        assert rule(M, N, tm, off) == want, (M, N, tm, off)
        seen[want] += 1
    assert min(seen) > 500
    assert not rule(704, 3200, 64, 3200) and not rule(538, 6145, 32, 6145 - 538) and rule(4096, 4096, 256, 0)


def test_ranges_of_what_a_mask_leaves():
    """Under a mask the ranges are those of the columns that the last row sees."""
    def ranges(b, M, K, N, off):
        p = make_problem(b, M, K, N, K, "f16", b_stride=(N * K, 1, K))
        return mcf.call_tiles(p, True, causal_offset=off)[1]
    assert ranges(33, 7, 192, 6282, 0) == ranges(5, 11, 96, 4305, -6) == ranges(23, 1, 64, 4604, -1) == ranges(3, 686, 192, 2789, -343) == 1
    assert ranges(33, 7, 192, 6282, 6282 - 7) == ranges(33, 7, 192, 6282, 10**6) > 1     # hides little, hides nothing
    for off in range(0, 8192, 317):                                                       # as for the columns alone
        assert ranges(32, 1, 128, 8192, off) == ranges(32, 1, 128, off + 1, off), off
    assert ranges(32, 1, 128, 8192, -5) == 1 and ranges(32, 1, 128, 8192, -10**6) == 1
