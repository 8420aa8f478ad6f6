"""Host-side checks that need no GPU: the C-ABI library loads and exports every symbol the
header declares, argument validation returns the documented codes before any launch, and the
tile picker's numbers agree with the paper's model as written out in oracle/perf_model.py."""
import ctypes
import os
import re

import pytest

import mcf_inputs as mi
import paper_2506_22169_amd as mcf
from oracle import perf_model as pm
from paper_2506_22169_amd.binding import Problem, Tiles, make_problem

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# machine constants the picker documents (MI355X): HBM and L2 bandwidth, MFMA peak, compute units
W_HBM, W_L2, P_MFMA, CUS, WAVE_CAP = 8.0e12, 32.0e12, 2.5e15, 256, 4
LDS_MAX = 160 * 1024


def _c_problem(w):
    return make_problem(w.batch, w.M, w.K, w.N, w.L, w.dtype,
                        b_stride=(w.N * w.K, 1, w.K) if w.softmax else None)


def test_library_exports_every_declared_symbol():
    header = open(os.path.join(ROOT, "include", "mcf.h")).read()
    declared = set(re.findall(r"\b(mcf_[a-z_]+)\s*\(", header))
    assert {"mcf_pick_tiles", "mcf_gemm_chain", "mcf_softmax_gemm_chain"} <= declared
    lib = mcf.load_library()
    for name in sorted(declared):
        assert getattr(lib, name) is not None, name
    assert mcf.status_string(0) == "MCF_OK"
    assert ctypes.sizeof(Problem) == 5 * 8 + 2 * 4 + 12 * 8
    assert ctypes.sizeof(Tiles) == 14 * 4 + 4 * 8 + 4 * 8


def test_validation_codes_without_a_launch():
    lib = mcf.load_library()
    p = make_problem(2, 64, 64, 64, 64, "f16")
    fake = [ctypes.c_void_p(4096 * (i + 1) * 1024) for i in range(4)]   # never dereferenced: every call below fails validation
    call = lambda prob, ptrs=fake: lib.mcf_gemm_chain(ctypes.byref(prob), *ptrs, None, None)
    assert lib.mcf_gemm_chain(None, *fake, None, None) == 1
    assert call(make_problem(2, 64, 48, 64, 48, "f16")) == 2                 # K, L not built
    assert call(make_problem(2, 64, 64, 64, 32, "f16")) == 2                 # K != L not built
    assert call(make_problem(2, -1, 64, 64, 64, "f16")) == 1                 # negative dimension
    assert call(make_problem(2, 64, 64, 60, 64, "f16")) == 3                 # packed rows of 60 are not 16-byte multiples
    assert call(make_problem(2, 64, 64, 60, 64, "f16", b_stride=(64 * 64, 64, 1))) == 2  # N-contiguous B needs N % 8 == 0
    assert call(make_problem(2, 64, 64, 64, 64, "f16", a_stride=(64 * 72, 72, 2))) == 2   # A not K-contiguous
    assert call(make_problem(2, 64, 64, 64, 64, "f16", a_stride=(64 * 68, 68, 1))) == 3   # row stride % 8
    assert call(make_problem(2, 64, 64, 64, 64, "f16", d_stride=(64 * 32, 32, 1))) == 1   # rows overlap
    # layout rules are also what the host-only picker checks (no launch can follow from it)
    tt = Tiles()
    pick = lambda prob: lib.mcf_pick_tiles(ctypes.byref(prob), 0, ctypes.byref(tt))
    assert call(make_problem(2, 64, 64, 64, 64, "f16", e_stride=(0, 64, 1))) == 1         # batches of E on top of one another
    assert pick(make_problem(2, 64, 64, 64, 64, "f16", e_stride=(63 * 64 + 56, 64, 1))) == 1  # ... overlapping by one piece
    assert pick(make_problem(2, 64, 64, 64, 64, "f16", e_stride=(63 * 64 + 64, 64, 1))) == 0  # ... exactly adjacent: fine
    assert pick(make_problem(1, 64, 64, 64, 64, "f16", e_stride=(0, 64, 1))) == 0         # one batch: its stride is not used
    assert pick(make_problem(2, 64, 64, 64, 64, "f16", a_stride=(0, 64, 1))) == 0         # a broadcast input is legal
    assert pick(make_problem(2, 64, 64, 64, 64, "f16", a_stride=(1 << 61, 64, 1))) == 2   # extent beyond 64-bit arithmetic
    assert call(make_problem(1 << 30, 64, 64, 64, 64, "f16", e_stride=(1 << 40, 64, 1))) == 2
    assert call(p, [ctypes.c_void_p(4096 + 2)] + fake[1:]) == 3                          # misaligned pointer
    assert call(p, [fake[3]] + fake[1:]) == 1                                            # E aliases A
    assert call(p, [None] + fake[1:]) == 1                                               # null pointer
    bad_out = make_problem(2, 64, 64, 64, 64, "f16")
    bad_out.out_dtype = 1                                                                # bf16 out of f16 in
    assert call(bad_out) == 2
    bad_out.in_dtype, bad_out.out_dtype = 2, 2                                           # fp32 inputs
    assert call(bad_out) == 2
    f32_out = make_problem(2, 64, 64, 64, 64, "f16")
    f32_out.out_dtype = 2                                                                # fp32 out: a layout the picker accepts
    assert pick(f32_out) == 0
    assert lib.mcf_causal_softmax_gemm_chain(ctypes.byref(make_problem(2, 64, 64, 0, 64, "f16")), ctypes.c_float(1.0),
                                             ctypes.c_int64(0), *fake, None, None) == 1   # softmax over nothing
    assert call(make_problem(0, 64, 64, 64, 64, "f16")) == 0                             # empty: no-op
    assert lib.mcf_softmax_gemm_chain(ctypes.byref(make_problem(2, 64, 64, 0, 64, "f16")), ctypes.c_float(1.0),
                                      *fake, None, None) == 1                            # softmax over nothing
    assert lib.mcf_softmax_gemm_chain(ctypes.byref(p), ctypes.c_float(float("nan")), *fake, None, None) == 1
    t = Tiles()
    assert lib.mcf_pick_tiles(ctypes.byref(p), 0, None) == 1
    assert lib.mcf_pick_tiles(ctypes.byref(make_problem(2, 64, 16, 64, 16, "f16")), 0, ctypes.byref(t)) == 2


_BUILT_PAPER_SHAPES = list(mi.PAPER_SHAPES)


@pytest.mark.parametrize("name", ["cfg1", "cfg2", "cfg3", "cfg4", "cfg5"] + _BUILT_PAPER_SHAPES)
def test_picker_terms_match_the_paper_model(name):
    """Every model term of every built variant, for T_L = L and for every smaller T_L that has
    kernels, equals eq. (2)-(5) evaluated by the oracle model for the tiling expression mhnk,
    and the picked variant is the feasible one with the smallest estimate."""
    w = mi.WORKLOADS[name] if name in mi.WORKLOADS else mi.PAPER_SHAPES[name]
    prob = _c_problem(w)
    shapes = mcf.list_variants(prob, w.softmax)
    assert len(shapes) >= (8 if w.K * w.L <= 128 * 128 else 3)
    dims = {"m": w.M, "n": w.N, "k": w.K, "h": w.L}
    pitch = lambda x: x if x % 32 == 0 else 1 << (x - 1).bit_length()   # LDS rows of whole 64-byte groups lie as they are
    tl_options = [w.L] + [tl for tl in (256, 128, 64, 32) if tl < w.L and w.L % tl == 0]
    best, n_ok = None, 0
    for tl in tl_options:
        # the arrangements built for (K, T_L): those of a problem whose L is T_L
        narrow = make_problem(w.batch, w.M, w.K, w.N, tl, w.dtype, b_stride=(w.N * w.K, 1, w.K) if w.softmax else None)
        for (mb, rg, ns, nj) in mcf.list_variants(narrow, w.softmax):
            t = mcf.eval_tiles(prob, mb, rg, ns, nj, tl=tl, softmax=w.softmax)
            assert (t.tm, t.tn, t.tl, t.waves) == (32 * mb * rg, 32 * ns * nj, tl, rg * ns)
            assert t.tk == (w.K if w.K <= 256 and (w.K, tl) != (256, 128) and (w.K, tl) != (256, 64) else 128)
            tiles = {"m": t.tm, "n": t.tn, "k": t.tk, "h": tl}
            units_per_block = (t.waves + 3) // 4
            # eq. (5) in rounds: a block takes min(waves, 4) of the four SIMDs of one of 256 compute units
            r = pm.estimate("mhnk", dims, tiles, w.batch, 2, W=W_HBM, P=P_MFMA,
                            n_units=CUS * WAVE_CAP // min(t.waves, WAVE_CAP), W_reread=W_L2, rounds=True)
            assert t.blocks == r["n_block"]
            assert t.compulsory_bytes == r["compulsory_bytes"] == w.compulsory_bytes
            assert t.model_bytes == r["model_bytes"]
            assert t.flops == r["flops"]
            assert t.t_mem_s == pytest.approx(r["t_mem"], rel=1e-12)
            assert t.t_comp_s == pytest.approx(r["t_comp"], rel=1e-12)
            assert t.alpha == pytest.approx(r["alpha"], rel=1e-12)
            assert t.t_est_s == pytest.approx(r["t_estm"], rel=1e-12)
            # eq. (1), split: LDS holds `stages` copies of the B and D tiles at least (plus the A tile in the last slot)
            padded = dict(tiles, k=pitch(t.tk), h=pitch(tl))
            bd = pm.shm_estm(padded, "BD") * 2
            a = pm.tile_elems("A", padded) * 2
            assert 2 <= t.stages <= 4     # (2 also where B and D have rings of their own)
            if t.tk < w.K:   # k loop: a ring slot holds the A + B chunk of a k step or the D tile
                ab = (pm.tile_elems("A", tiles) + pm.tile_elems("B", tiles)) * 2
                assert t.lds_bytes >= t.stages * max(ab, pm.tile_elems("D", tiles) * 2)
            else:
                assert t.lds_bytes >= (t.stages - 1) * bd + max(bd, a)
            ok = (t.lds_bytes <= LDS_MAX and t.scratch_bytes == 0 and t.vgpr_est <= 512 // units_per_block
                  and pm.padding_ok(w.M, t.tm) and pm.padding_ok(w.N, t.tn))
            assert ok == (t.feasible and pm.padding_ok(w.M, t.tm) and pm.padding_ok(w.N, t.tn))
            n_ok += ok
            if ok and (best is None or t.t_est_s < best.t_est_s * (1 - 1e-12)):
                best = t
    cands = mcf.list_candidates(prob, w.softmax)
    assert len(cands) == n_ok                      # the candidate list is exactly the feasible set
    assert cands[0].tl == w.L and all(c.tl <= w.L and w.L % c.tl == 0 for c in cands)
    picked = mcf.pick_tiles(prob, w.softmax)
    assert best is not None
    assert picked.t_est_s == pytest.approx(best.t_est_s, rel=1e-12)
    assert picked.scratch_bytes == 0 and picked.lds_bytes <= LDS_MAX
    assert pm.padding_ok(w.M, picked.tm) and pm.padding_ok(w.N, picked.tn)


def test_shapes_without_kernels_are_refused():
    """(K, L) that no group covers have no built kernels: the picker says so instead of
    returning something that cannot run.  K = 512, 1024 (G5, G6) are served by the kernels
    with a k loop of T_K = 128."""
    lib = mcf.load_library()
    t = Tiles()
    assert lib.mcf_pick_tiles(ctypes.byref(make_problem(16, 256, 48, 256, 48, "f16")), 1, ctypes.byref(t)) == 2
    assert lib.mcf_pick_tiles(ctypes.byref(make_problem(1, 512, 192, 512, 64, "f16")), 0, ctypes.byref(t)) == 2  # 192 = 1.5 chunks
    assert lib.mcf_pick_tiles(ctypes.byref(make_problem(1, 512, 512, 512, 32, "f16")), 0, ctypes.byref(t)) == 2  # no k-loop group with L = 32
    for name in ("G5", "G6"):
        w = mi.PAPER_SHAPES[name]
        assert lib.mcf_pick_tiles(ctypes.byref(_c_problem(w)), 0, ctypes.byref(t)) == 0
        assert t.tk == 128 and t.tk < w.K and w.L % t.tl == 0


def test_register_estimate_tracks_the_compiler():
    """The register form of eq. (1): within 45 % below / 60 % above what the compiler allocated
    where registers are scarce (blocks of eight waves; with four the allocator spends freely what the
    block leaves unused),
    and every variant the estimate admits under its register cap compiled without spilling,
    with at most a few exceptions (the analogue of the paper's estimate-vs-lowering check)."""
    total = wrong = 0
    for dtype in ("f16", "bf16"):
        for K, L in ((32, 32), (64, 64), (128, 128), (64, 128), (128, 64), (64, 256), (256, 256), (80, 80)):
            for softmax in (False, True):
                prob = make_problem(4, 1024, K, 1024, L, dtype, b_stride=(1024 * K, 1, K) if softmax else None)
                for shape in mcf.list_variants(prob, softmax):
                    t = mcf.eval_tiles(prob, *shape, softmax=softmax)
                    cap = 512 // ((t.waves + 3) // 4)
                    assert t.vgpr_used > 0
                    total += 1
                    admitted = t.vgpr_est <= cap
                    if admitted != (t.scratch_bytes == 0):
                        wrong += 1
                    if t.scratch_bytes == 0 and t.vgpr_used < cap and t.waves > 4:   # two waves per SIMD: registers are scarce
                        assert 0.55 * t.vgpr_used <= t.vgpr_est <= 1.6 * t.vgpr_used, (dtype, K, L, softmax, shape)
    assert total >= 150 and wrong <= 0.1 * total


def test_rule3_fallback_and_ragged_shapes():
    # M smaller than every tile: Rule 3 cannot hold, the picker still returns a covering variant
    t = mcf.pick_tiles(make_problem(1, 16, 64, 64, 64, "f16"))
    assert t.tm >= 32 and t.blocks == 1
    # non power of two: padding ratio below 5 %
    t = mcf.pick_tiles(make_problem(4, 1000, 64, 1000, 64, "f16"))
    assert pm.padding_ok(1000, t.tm) and pm.padding_ok(1000, t.tn)
    # the number of blocks drives alpha: a single small batch prefers the smallest m-tile
    t = mcf.pick_tiles(make_problem(1, 1024, 64, 128, 64, "f16"))
    assert t.tm == 32


def test_three_gemm_chain_host_side():
    """Arrangements built for the three-GEMM chain, for (K, L, P) in {(64,64,64), (128,128,128), (64,128,128),
    (128,64,64), (64,64,128)}: a subset of those of the two-GEMM chain, with and without a split of n across
    waves where P = L (the combine of the product reuses the layout of E), without one where P != L; the
    default pick is one of them, one with the smallest two-GEMM estimate; other shapes are refused."""
    for K, L, P in ((64, 64, 64), (128, 128, 128), (64, 128, 128), (128, 64, 64), (64, 64, 128)):
        for dtype in ("f16", "bf16"):
            for softmax in (False, True):
                prob = make_problem(8, 1024, K, 1024, L, dtype, b_stride=(1024 * K, 1, K) if softmax else None)
                shapes = mcf.list_variants3(prob, P, softmax)
                assert len(shapes) >= 4
                assert {s[2] for s in shapes} >= ({1, 2} if P == L else {1}) and (P == L or {s[2] for s in shapes} == {1})
                assert set(shapes) <= set(mcf.list_variants(prob, softmax))
                t = mcf.pick_tiles3(prob, P, softmax)
                assert (t.mb, t.rg, t.ns, t.nj) in shapes
                ests = {s: mcf.eval_tiles(prob, *s, softmax=softmax).t_est_s for s in shapes}
                assert t.t_est_s == min(ests.values())
    prob = make_problem(8, 1024, 64, 1024, 64, "f16")
    assert mcf.list_variants3(prob, 32, False) == []
    with pytest.raises(mcf.McfError) as e:
        mcf.pick_tiles3(prob, 256, False)
    assert e.value.status == 2
    with pytest.raises(mcf.McfError) as e:
        mcf.pick_tiles3(make_problem(8, 1024, 32, 1024, 32, "f16"), 32, False)
    assert e.value.status == 2
