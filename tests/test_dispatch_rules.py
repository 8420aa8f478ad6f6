"""What a call without an arrangement runs, on the host: which calls split n, into how much, and
that a split call asks for the workspace its ranges need."""
import ctypes

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
    assert _workspace(5, 953, 64, 3696, 64, "f16", 0, P=128, out_f32=out_f32) >= 2
    assert _workspace(1, 209, 96, 3003, 96, "f16", 2, out_f32=out_f32) >= 2


def test_calls_that_do_not_split():
    assert _workspace(64, 512, 64, 512, 64) == 0            # a block for every compute unit
    assert _workspace(1, 1024, 64, 128, 64) == 0            # one n-tile
    assert _workspace(4, 128, 64, 512, 64, "f16", 1) == 0   # nothing to win: a few n-tiles
    assert _workspace(32, 1, 128, 8192, 128, "bf16", 1, n_split=1) == 0
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
