"""Softmax chains whose scores outgrow the reference that the pipelined loops leave standing: by a
little, past fp16, past the range of the exponential, in tiles of either parity, once and again and
again, and rows that see nothing for some tiles; against the fp64 oracle.  Needs an MI355X."""
import numpy as np
import pytest
import torch

import mcf_inputs as mi
import oracle
import paper_2506_22169_amd as mcf

from gpu_util import TOL, device_inputs, to_host64

pytestmark = pytest.mark.gpu

# K = L, dtype, tiles: one or two row sets a wave, one or two waves across n, one or two blocks a compute unit
KERNELS = [(64, "f16", (1, 8, 1, 2)), (64, "bf16", (2, 4, 2, 1)), (64, "f16", (1, 4, 1, 1)), (128, "bf16", (1, 8, 1, 2)),
           (128, "f16", (1, 8, 1, 1)), (96, "bf16", (1, 8, 1, 1)), (128, "bf16", (1, 2, 2, 1))]
# factor on the keys from a column on: (column, factor) pairs
GROWTH = [[(200, 4.0)], [(263, 60.0)], [(130, 3.0), (200, 9.0), (264, 27.0), (390, 60.0)], [(129, 0.02), (390, 30.0)]]


def _grown(w, steps):
    x = mi.make_inputs(w)
    f = np.ones(w.N)
    for col, by in steps:
        f[col:] = by
    x["b_bits"] = mi.to_bits(mi.from_bits(x["b_bits"], w.dtype) * f[None, :, None], w.dtype)
    x["B"] = mi.from_bits(x["b_bits"], w.dtype).transpose(0, 2, 1)
    return x


def _compare(got, ref, what):
    assert np.isfinite(got).all(), what
    err, scale = np.max(np.abs(got - ref)), np.max(np.abs(ref))
    assert err <= TOL * scale, f"{what}: {err:.4g} > {TOL} * {scale:.4g}"


@pytest.mark.parametrize("kernel", KERNELS, ids=str)
@pytest.mark.parametrize("steps", GROWTH, ids=lambda g: "_".join(f"{c}x{f}" for c, f in g))
def test_growing_scores(kernel, steps):
    K, dtype, tiles = kernel
    w = mi.make_problem(2, 300, K, 531, K, dtype, True, "normal", seed=9400 + K)
    x = _grown(w, steps)
    A, B, D = device_inputs(w, x)
    print("case growing", kernel, steps, flush=True)
    got = to_host64(mcf.softmax_gemm_chain(A, B, D, w.scale, tiles=tiles), dtype)
    _compare(got, oracle.chain(x["A"], x["B"], x["D"], softmax=True, scale=w.scale), (kernel, steps))


@pytest.mark.parametrize("off", [231, 0, -70], ids=lambda o: f"off{o}")
@pytest.mark.parametrize("kernel", KERNELS, ids=str)
def test_growing_scores_under_a_mask(kernel, off):
    K, dtype, tiles = kernel
    w = mi.make_problem(2, 600, K, 531, K, dtype, True, "normal", seed=9500 + K)
    x = _grown(w, [(130, 3.0), (263, 40.0)])
    A, B, D = device_inputs(w, x)
    print("case growing causal", kernel, off, flush=True)
    got = to_host64(mcf.causal_softmax_gemm_chain(A, B, D, w.scale, off, tiles=tiles), dtype)
    _compare(got, oracle.chain_causal(x["A"], x["B"], x["D"], scale=w.scale, causal_offset=off), (kernel, off))
    assert not got[:, np.arange(w.M) + off < 0].any()


def test_results_do_not_depend_on_the_other_rows():
    """A row whose scores outgrow the reference sends its wave the other way: its neighbours get what
    they get without it, up to the rounding of the 16-bit P."""
    w = mi.make_problem(1, 256, 64, 531, 64, "f16", True, "normal", seed=9600)
    x = mi.make_inputs(w)
    a = mi.from_bits(x["a_bits"], "f16")
    a[0, 7] *= 40.0
    y = dict(x, a_bits=mi.to_bits(a, "f16"))
    calm, wild = (to_host64(mcf.softmax_gemm_chain(*device_inputs(w, z), w.scale, tiles=(1, 8, 1, 2)), "f16") for z in (x, y))
    keep = np.arange(256) != 7
    # half an ulp of every p on either side, weighed with at most max|D|, and half an ulp of the result on either side
    assert np.max(np.abs(calm[0, keep] - wild[0, keep])) <= 2.0**-10 * (np.max(np.abs(x["D"])) + np.max(np.abs(calm)))


@pytest.mark.parametrize("kernel", [k for k in KERNELS if k[1] == "bf16"], ids=str)
@pytest.mark.parametrize("col", [140, 300, 530])
@pytest.mark.parametrize("exponent", [117, -118])
def test_sums_stay_within_fp32(kernel, col, exponent):
    """One score 2^11 above the reference of the first tile, and D at 2^118: a sum of p D with p of 2^11 is
    beyond fp32 while every result is at most max|D|.  p may not grow past 2^8.  And D at 2^-117: nor may
    p be so small that the products are lost."""
    K, dtype, tiles = kernel
    w = mi.make_problem(1, 300, K, 531, K, dtype, True, "normal", seed=9650 + K)
    x = mi.make_inputs(w)
    a, b = np.zeros((1, 300, K)), np.zeros((1, 531, K))
    a[:, :, 0], b[:, col, 0] = 8.0, 0.95
    d = mi.from_bits(x["d_bits"], dtype)
    d = np.clip(d, -2.0, 2.0) * 2.0**exponent
    bits = {"a_bits": mi.to_bits(a, dtype), "b_bits": mi.to_bits(b, dtype), "d_bits": mi.to_bits(d, dtype)}
    A, B, D = device_inputs(w, dict(x, **bits))
    print("case fp32 range", kernel, col, exponent, flush=True)
    got = to_host64(mcf.softmax_gemm_chain(A, B, D, 1.0, tiles=tiles), dtype)
    ref = oracle.chain(*(mi.from_bits(bits[k], dtype) if k != "b_bits" else mi.from_bits(bits[k], dtype).transpose(0, 2, 1)
                         for k in ("a_bits", "b_bits", "d_bits")), softmax=True, scale=1.0)
    _compare(got, ref, (kernel, col, exponent))


@pytest.mark.parametrize("kernel", KERNELS, ids=str)
def test_nan_rows_stay_by_themselves(kernel):
    """A row of NaN scores is NaN, and the other rows of its wave are what they are without it, to the bit: such
    a row moves no other row's reference and costs no second pass over a tile."""
    K, dtype, tiles = kernel
    w = mi.make_problem(1, 256, K, 531, K, dtype, True, "normal", seed=9680 + K)
    x = mi.make_inputs(w)
    A, B, D = device_inputs(w, x)
    calm = to_host64(mcf.softmax_gemm_chain(A, B, D, w.scale, tiles=tiles), dtype)
    A[0, 9, 0] = float("nan")
    print("case nan rows", kernel, flush=True)
    got = to_host64(mcf.softmax_gemm_chain(A, B, D, w.scale, tiles=tiles), dtype)
    keep = np.arange(256) != 9
    assert np.isnan(got[0, 9]).all()
    assert np.array_equal(got[0, keep], calm[0, keep])
