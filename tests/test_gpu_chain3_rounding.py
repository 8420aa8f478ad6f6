"""Chains of three GEMMs whose E is small against its parts: E is rounded once, before the third GEMM, so
that parts of the n range that cancel, or that are beyond fp16, must not be rounded on their own.
Calls without tiles, where the library chooses.  Needs an MI355X."""
import numpy as np
import pytest
import torch

import mcf_inputs as mi
import oracle
import paper_2506_22169_amd as mcf

from gpu_util import TOL, to_device, to_host64

pytestmark = pytest.mark.gpu

# (batch, M, K, N, L, P) and the columns of a run: a few blocks with a long n range, in one wave across n; a ragged N that
# pads least with 32 columns; and waves across n by the model's own pick, each of which gets both signs
CASES = [((5, 953, 64, 4096, 64, 128), 64), ((5, 953, 64, 4096, 64, 128), 2048), ((6, 827, 64, 2200, 64, 128), 32),
         ((20, 827, 128, 1112, 64, 64), 32), ((20, 827, 128, 1112, 64, 64), 64), ((1, 128, 64, 4096, 64, 64), 2048)]


def _alternating(shape, run, top, noise, step):
    """Rows of D of one sign for `run` columns of C, then of the other, on a grid of `step`, and noise that does not cancel."""
    b, M, K, N, L, P = shape
    rng = np.random.default_rng(9800 + run)
    sign = np.where((np.arange(N) // run) % 2 == 0, 1.0, -1.0)[:, None]
    base = np.round(rng.uniform(top / 2, top, (1, L)) / step) * step
    return np.broadcast_to(sign * base, (b, N, L)) + np.round(rng.uniform(-noise, noise, (b, N, L)) / step) * step


@pytest.mark.parametrize("shape,run", CASES, ids=str)
@pytest.mark.parametrize("softmax", [False, True])
def test_parts_of_e_that_cancel(shape, run, softmax):
    b, M, K, N, L, P = shape
    if softmax:  # equal weights: E is the mean of D, about 1, of parts of 256 to 512
        a, bt, d = np.zeros((b, M, K)), np.ones((b, N, K)), _alternating(shape, run, 512.0, 32.0, 0.5)
    else:        # parts of E up to 10^5, beyond fp16, E itself some hundreds
        rng = np.random.default_rng(9850)
        a, bt, d = rng.uniform(0, 1, (b, M, K)), np.full((b, N, K), 0.5), _alternating(shape, run, 8.0, 0.5, 1 / 64)
    half = N // (2 * run) * 2 * run  # whole pairs of runs cancel; the rest is left out
    d[:, half:] = 0.0
    f = mi.draw(9870, 4, (b, L, P), "uniform")
    bits = [mi.to_bits(t, "f16") for t in (a, bt, d, f)]
    a, bt, d, f = (mi.from_bits(t, "f16") for t in bits)
    A, Bt, D, F = (to_device(t, "f16") for t in bits)
    print("case cancelling", shape, run, softmax, flush=True)
    got = to_host64(mcf.gemm_chain3(A, Bt.transpose(1, 2) if softmax else Bt.transpose(1, 2).contiguous(), D, F, scale=1.0 if softmax else None), "f16")
    ref = oracle.chain3(a, bt.transpose(0, 2, 1), d, f, softmax=softmax, scale=1.0)
    err, scale = np.max(np.abs(got - ref)), np.max(np.abs(ref))
    assert np.isfinite(got).all() and err <= TOL * scale, f"{shape} {run}: {err:.4g} > {TOL} * {scale:.4g}"
