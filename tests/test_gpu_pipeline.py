"""The softmax pipeline's rings (B two tiles ahead of D, some with one more tile in flight, the first D tiles before the loop): every
arrangement over one to a few n-tiles, whole and ragged, and under a mask that ends the loop before the last column (no load may be
on its way when the ring's space is used again)."""
import numpy as np
import pytest

import mcf_inputs as mi
import oracle
import paper_2506_22169_amd as mcf
from gpu_util import TOL, device_inputs, to_host64
from paper_2506_22169_amd.binding import list_variants, make_problem

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _err(E, ref, dtype):
    return np.max(np.abs(to_host64(E, dtype) - ref)) / np.max(np.abs(ref))


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("KL", [(32, 32), (64, 64), (80, 80), (96, 96), (128, 128), (160, 160), (192, 192), (256, 256), (64, 128), (128, 64)])
def test_every_arrangement_masked_and_not(KL, dtype):
    K, L = KL
    M = 290
    for N, offsets in ((24, (None,)), (96, (None, -200)), (264, (None, -27)), (392, (None, 0, 102)), (640, (None, 0, 350))):
        w = mi.make_problem(2, M, K, N, L, dtype, True, "normal", seed=4100 + K + L + N)
        x = mi.make_inputs(w)
        A, B, D = device_inputs(w, x)
        for off in offsets:
            ref = (oracle.chain(x["A"], x["B"], x["D"], softmax=True, scale=w.scale) if off is None
                   else oracle.chain_causal(x["A"], x["B"], x["D"], w.scale, off))
            for tiles in list_variants(make_problem(2, M, K, N, L, dtype, b_stride=(N * K, 1, K)), True):
                print(f"case K={K} L={L} {dtype} N={N} offset={off} tiles={tiles}", flush=True)
                E = (mcf.softmax_gemm_chain(A, B, D, w.scale, tiles=tiles) if off is None
                     else mcf.causal_softmax_gemm_chain(A, B, D, w.scale, off, tiles=tiles))
                torch.cuda.synchronize()
                assert _err(E, ref, dtype) <= TOL, (N, off, tiles)
