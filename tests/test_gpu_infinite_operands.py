"""Infinities in D in a ragged last n-tile: a slice of 32 columns that has none of the tile's must not meet D, whose rows beyond N are
stood in for by row N - 1 (0 x Inf would turn an infinite element into a NaN).  Needs an MI355X."""
import numpy as np
import pytest
import torch

import mcf_inputs as mi
import oracle
import paper_2506_22169_amd as mcf

from gpu_util import TOL, device_inputs, to_host64
from paper_2506_22169_amd.binding import call_tiles, list_variants, make_problem

pytestmark = pytest.mark.gpu


def _check(w, x, run, L, weight_sign):
    """run(D) with infinities of both signs in row N - 1 of D: infinite there, as it was in every other column."""
    _, _, D = device_inputs(w, x)
    Dinf = D.clone()
    Dinf[:, w.N - 1, 3] = float("inf")
    Dinf[:, w.N - 1, L - 1] = -float("inf")
    finite, got = to_host64(run(D), w.dtype), to_host64(run(Dinf), w.dtype)
    assert np.array_equal(got[:, :, 3], weight_sign * np.inf) and np.array_equal(got[:, :, L - 1], -weight_sign * np.inf)
    keep = [c for c in range(L) if c not in (3, L - 1)]
    assert np.array_equal(got[:, :, keep], finite[:, :, keep])
    return finite


def _last_column_sign(w, x):
    """The weight of row N - 1: P > 0 (softmax) or the last column of C, whose sign decides."""
    if w.softmax:
        return np.ones((w.batch, w.M))
    return np.sign(x["A"] @ x["B"][:, :, w.N - 1:])[..., 0]


# with a k loop: N is a multiple of a wave's own columns (32 nj) and not of the n-tile
@pytest.mark.parametrize("tiles,N,L", [((1, 1, 4, 1), 96, 64), ((1, 1, 4, 1), 160, 128), ((1, 2, 2, 1), 32, 64), ((1, 1, 2, 2), 64, 64),
                                       ((1, 1, 8, 1), 288, 128), ((2, 1, 4, 1), 224, 64)], ids=str)
@pytest.mark.parametrize("softmax", [False, True])
def test_infinite_last_row_of_d(tiles, N, L, softmax):
    w = mi.make_problem(2, 70, 384, N, L, "f16", softmax, "normal" if softmax else "uniform", seed=9700 + N)
    x = mi.make_inputs(w)
    A, B, D = device_inputs(w, x)
    print("case infinite", tiles, N, L, softmax, flush=True)
    run = lambda d: mcf.softmax_gemm_chain(A, B, d, w.scale, tiles=tiles) if softmax else mcf.gemm_chain(A, B, d, tiles=tiles)
    finite = _check(w, x, run, L, _last_column_sign(w, x))
    ref = oracle.chain(x["A"], x["B"], x["D"], softmax=softmax, scale=w.scale)
    assert np.max(np.abs(finite - ref)) <= TOL * np.max(np.abs(ref))


@pytest.mark.parametrize("KL", [(32, 32), (64, 64), (80, 80), (96, 96), (128, 128), (160, 160), (256, 256)], ids=str)
@pytest.mark.parametrize("softmax", [False, True])
def test_infinite_last_row_of_d_whole_k(KL, softmax):
    """Every arrangement with the whole K on chip: one ragged tile alone, whole tiles before it, waves and slices without a column of it."""
    K, L = KL
    for N in (32, 160, 352, 800):
        w = mi.make_problem(2, 70, K, N, L, "bf16", softmax, "normal" if softmax else "uniform", seed=9800 + N + K)
        x = mi.make_inputs(w)
        A, B, _ = device_inputs(w, x)
        sign = _last_column_sign(w, x)
        for tiles in list_variants(make_problem(2, 70, K, N, L, "bf16", b_stride=(N * K, 1, K) if softmax else None), softmax):
            print("case infinite", tiles, N, KL, softmax, flush=True)
            _check(w, x, lambda d: mcf.softmax_gemm_chain(A, B, d, w.scale, tiles=tiles) if softmax else mcf.gemm_chain(A, B, d, tiles=tiles), L, sign)


# calls without tiles: a decode call in ranges of n, two slices a wave where n-tiles of 32 columns would fit N
@pytest.mark.parametrize("softmax,b,M,N,K", [(True, 32, 1, 2080, 128), (True, 20, 4, 1056, 96), (False, 40, 1000, 800, 96), (True, 40, 1216, 1312, 128)])
def test_infinite_last_row_of_d_in_calls_without_tiles(softmax, b, M, N, K):
    w = mi.make_problem(b, M, K, N, K, "bf16", softmax, "normal" if softmax else "uniform", seed=9900 + N)
    x = mi.make_inputs(w)
    A, B, _ = device_inputs(w, x)
    t, ranges = call_tiles(make_problem(b, M, K, N, K, "bf16", b_stride=(N * K, 1, K) if softmax else None), softmax)
    print("case infinite", (t.mb, t.rg, t.ns, t.nj, t.tl), ranges, (b, M, N, K), flush=True)
    assert N % t.tn != 0
    _check(w, x, lambda d: mcf.softmax_gemm_chain(A, B, d, w.scale) if softmax else mcf.gemm_chain(A, B, d), K, _last_column_sign(w, x))


@pytest.mark.parametrize("KLP", [(64, 64, 64), (128, 128, 128)], ids=str)
@pytest.mark.parametrize("N", [32, 160, 352])
def test_infinite_last_row_of_d_of_three_gemms(KLP, N):
    """One infinite column of E makes every element of E . F infinite with the sign of its row of F."""
    K, L, P = KLP
    w = mi.make_problem(2, 70, K, N, L, "bf16", True, "normal", seed=9950 + N)
    x = mi.make_inputs(w)
    A, B, D = device_inputs(w, x)
    F = torch.where(torch.arange(2 * L * P, device="cuda").reshape(2, L, P) % 3 == 0, -0.5, 0.25).to(torch.bfloat16)
    D[:, N - 1, 3] = float("inf")
    want = np.broadcast_to(np.sign(F[:, 3:4, :].double().cpu().numpy()) * np.inf, (2, 70, P))
    for tiles in mcf.list_variants3(make_problem(2, 70, K, N, L, "bf16", b_stride=(N * K, 1, K)), P, True):
        print("case infinite", tiles, N, KLP, flush=True)
        assert np.array_equal(to_host64(mcf.gemm_chain3(A, B, D, F, scale=w.scale, tiles=tiles), "bf16"), want), tiles
