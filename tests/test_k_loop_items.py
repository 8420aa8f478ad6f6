"""Kernels with a k loop whose ring items are half a chunk deep ((1,1,8,1) and (1,1,4,2) of plain chains with L = 64): the first and the
last items, one n-tile and several, both layouts of B, ranges of n."""
import numpy as np
import pytest

import mcf_inputs as mi
import oracle
import paper_2506_22169_amd as mcf
from gpu_util import TOL, device_inputs, to_host64
from paper_2506_22169_amd import binding

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("K", [256, 384, 1024])
@pytest.mark.parametrize("tiles", [(1, 1, 8, 1, 64), (1, 1, 4, 2, 64)], ids=str)
def test_half_chunk_items(tiles, K, dtype):
    for N, L in ((8, 64), (264, 64), (520, 128)):
        w = mi.make_problem(2, 75, K, N, L, dtype, False, "uniform", seed=6100 + K + N)
        x = mi.make_inputs(w)
        A, B, D = device_inputs(w, x)
        ref = oracle.chain(x["A"], x["B"], x["D"])
        for b in (B.contiguous(), B.transpose(1, 2).contiguous().transpose(1, 2)):
            for ranges in (1, 2):
                print(f"case K={K} N={N} L={L} {dtype} tiles={tiles} strides={b.stride()} ranges={ranges}", flush=True)
                E = binding._call(0, 1.0, 0, A, b, D, None, None, tiles, None, ranges)
                torch.cuda.synchronize()
                assert np.max(np.abs(to_host64(E, dtype) - ref)) <= TOL * np.max(np.abs(ref)), (N, L, ranges)
