"""Infinities in D of the chains with a k loop: in a ragged last n-tile the waves that have no column of it
must not touch D, whose rows beyond N are stood in for by row N - 1 (0 x Inf would turn an infinite
element into a NaN).  Needs an MI355X."""
import numpy as np
import pytest
import torch

import mcf_inputs as mi
import oracle
import paper_2506_22169_amd as mcf

from gpu_util import TOL, device_inputs, to_host64

pytestmark = pytest.mark.gpu


# N is a multiple of a wave's own columns (32 nj) and not of the n-tile: one wave at least has none in the last tile
@pytest.mark.parametrize("tiles,N,L", [((1, 1, 4, 1), 96, 64), ((1, 1, 4, 1), 160, 128), ((1, 2, 2, 1), 32, 64), ((1, 1, 2, 2), 64, 64),
                                       ((1, 1, 8, 1), 288, 128), ((2, 1, 4, 1), 224, 64)], ids=str)
@pytest.mark.parametrize("softmax", [False, True])
def test_infinite_last_row_of_d(tiles, N, L, softmax):
    w = mi.make_problem(2, 70, 384, N, L, "f16", softmax, "normal" if softmax else "uniform", seed=9700 + N)
    x = mi.make_inputs(w)
    A, B, D = device_inputs(w, x)
    print("case infinite", tiles, N, L, softmax, flush=True)
    run = lambda d: mcf.softmax_gemm_chain(A, B, d, w.scale, tiles=tiles) if softmax else mcf.gemm_chain(A, B, d, tiles=tiles)
    Dinf = D.clone()
    Dinf[:, N - 1, 3] = float("inf")
    Dinf[:, N - 1, L - 1] = -float("inf")
    finite, got = to_host64(run(D), "f16"), to_host64(run(Dinf), "f16")
    # the weight of row N - 1: P > 0 (softmax) or the last column of C, whose sign decides
    sign = np.ones((2, 70)) if softmax else np.sign(x["A"] @ x["B"][:, :, N - 1:])[..., 0]
    assert np.array_equal(got[:, :, 3], sign * np.inf) and np.array_equal(got[:, :, L - 1], -sign * np.inf)
    keep = [c for c in range(L) if c not in (3, L - 1)]
    assert np.array_equal(got[:, :, keep], finite[:, :, keep])
    ref = oracle.chain(x["A"], x["B"], x["D"], softmax=softmax, scale=w.scale)
    assert np.max(np.abs(finite - ref)) <= TOL * np.max(np.abs(ref))
