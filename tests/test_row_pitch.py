"""LDS rows of K, L that are multiples of 32 but no powers of two lie at their own pitch (96: 192 bytes, 160: 320, 192: 384), with
the swizzle inside the largest power of two that divides it; K = 256 spans two swizzle periods."""
import os
import subprocess

import numpy as np
import pytest

import mcf_inputs as mi
import oracle
import paper_2506_22169_amd as mcf
from paper_2506_22169_amd.binding import call_tiles, list_variants, make_problem

SIZES = (96, 160, 192, 256)


@pytest.mark.parametrize("N,nj", [(776, 2), (520, 2), (456, 2), (136, 1), (200, 1)])
def test_two_slices_where_they_pad_little(N, nj):
    """Eight waves across m of a plain chain: n-tiles of 64 columns where they pad N by an eighth at most."""
    for K in (64, 96, 128):
        t, ranges = call_tiles(make_problem(40, 1000, K, N, K, "bf16"))
        if (t.mb, t.rg, t.ns) != (1, 8, 1):
            continue
        assert ranges == 1 and t.nj == (2 if 8 * (-N % 64) <= N else 1) == nj, (K, N)
    t, _ = call_tiles(make_problem(40, 1000, 96, 776, 96, "bf16"))
    assert (t.mb, t.rg, t.ns, t.nj) == (1, 8, 1, 2)


BLOCKS = """
#include <initializer_list>

#include "mcf_geometry.h"
using namespace mcf;
int main() {
    for (int rb : {64, 128, 192, 256, 320, 384, 512})
        for (int row = 0; row < 64; ++row)
            for (int u = 0; u < 4; ++u)
                for (int block = 0; block < rb / 64; ++block) {
                    const int first = row * rb + 16 * (u ^ swz_tr(rb, row)), want = row * rb + 16 * ((4 * block + u) ^ swz_tr(rb, row));
                    if ((first ^ tr_block_xor(rb, block)) + tr_block_add(rb, block) != want) return 1;
                    if (swz_tr(rb, row) != swz_tr(rb, row + 4)) return 2;
                }
    return 0;
}
"""


def test_blocks_of_a_row_for_every_pitch(tmp_path):
    """The third GEMM's reads of F find every 64-byte block of a row where the loads have put it, also for pitches that no kernel has."""
    (tmp_path / "blocks.cpp").write_text(BLOCKS)
    csrc = os.path.join(os.path.dirname(os.path.abspath(mcf.__file__)), "csrc")
    subprocess.run(["g++", "-std=c++17", "-I", csrc, str(tmp_path / "blocks.cpp"), "-o", str(tmp_path / "blocks")], check=True)
    assert subprocess.run([str(tmp_path / "blocks")]).returncode == 0


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("softmax", [False, True])
@pytest.mark.parametrize("K", SIZES)
def test_own_pitch_in_the_other_layout_of_b(K, softmax, dtype):
    """Every arrangement, plain chains with B as [b,N,K] and softmax chains with B as [b,K,N], one column over a tile and eight
    short of one; and every arrangement's stores end with the row (partial last blocks of several waves)."""
    import torch

    from gpu_util import TOL, device_inputs, to_host64
    for N in (72, 184):
        w = mi.make_problem(2, 70, K, N, K, dtype, softmax, "normal" if softmax else "uniform", seed=300 + K + N)
        x = mi.make_inputs(w)
        A, B, D = device_inputs(w, x)
        B = B.contiguous() if softmax else B.transpose(1, 2).contiguous().transpose(1, 2)
        ref = oracle.chain(x["A"], x["B"], x["D"], softmax=softmax, scale=w.scale)
        prob = make_problem(2, 70, K, N, K, dtype, b_stride=None if softmax else (N * K, 1, K))
        for tiles in list_variants(prob, softmax):
            print(f"case K={K} N={N} {dtype} softmax={softmax} tiles={tiles}", flush=True)
            wide = torch.full((2, 70, K + 32), 7.0, dtype=A.dtype, device="cuda")   # columns beyond the row must stay
            out = wide[:, :, :K]
            E = mcf.softmax_gemm_chain(A, B, D, w.scale, out=out, tiles=tiles) if softmax else mcf.gemm_chain(A, B, D, out=out, tiles=tiles)
            torch.cuda.synchronize()
            assert np.max(np.abs(to_host64(E, dtype) - ref)) <= TOL * np.max(np.abs(ref)), tiles
            assert bool((wide[:, :, K:] == 7.0).all()), tiles
