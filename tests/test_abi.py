"""The shared library loads without a GPU and exports every symbol the headers declare;
argument errors are reported through ax_status without touching a device."""
import ctypes
import glob
import os
import re

import numpy as np
import pytest

from paper_2605_10380_amd import binding as B
from paper_2605_10380_amd import inputs as I

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def declared_symbols():
    names = set()
    for h in glob.glob(os.path.join(ROOT, "include", "*.h")):
        text = re.sub(r"/\*.*?\*/", "", open(h).read(), flags=re.S)
        names |= set(re.findall(r"\b(ax_[a-z0-9_]+)\s*\(", text))
    return names


def test_every_declared_symbol_is_exported():
    syms = declared_symbols()
    assert {"ax_kv_alloc", "ax_kv_fork", "ax_extend", "ax_verify", "ax_kv_free", "ax_kv_truncate",
            "ax_extend_batch", "ax_model_create", "ax_pool_create"} <= syms
    lib = ctypes.CDLL(B.LIB_PATH)
    for s in sorted(syms):
        assert hasattr(lib, s), f"{s} declared in include/ but not exported"


def test_binding_has_the_same_names():
    for s in declared_symbols() - {"ax_last_error"}:
        assert hasattr(B, s), s


def test_config_validation_without_gpu():
    sh = I.SHAPES["1b"]
    good = B.make_config(sh, 8192, 256)
    assert B.ax_workspace_bytes(good) > 0
    for field, val in [("n_layers", 0), ("n_q_heads", 7), ("dtype", 3), ("max_tokens", 0), ("head_dim", 96),
                       ("d_ff", 100), ("vocab", 1000)]:
        bad = B.make_config(sh, 8192, 256)
        setattr(bad, field, val)
        assert B.ax_workspace_bytes(bad) == 0, field
        with pytest.raises(B.AxError):
            B.ax_pool_create(bad, 0, 1 << 30)
    with pytest.raises(B.AxError) as e:
        B.ax_pool_create(good, 0, 1 << 30, block_tokens=32)
    assert e.value.status == B.AX_ERR_UNSUPPORTED
    with pytest.raises(B.AxError) as e:
        B.ax_pool_create(good, 0, 1000)
    assert e.value.status == B.AX_ERR_OOM
    with pytest.raises(B.AxError):
        B.ax_model_create(good, {k: 0 for k in ("tok_emb", "lm_head", "final_norm")} |
                          {k: [0] * sh.n_layers for k in ("wqkv", "wo", "w_gate", "w_up", "w_down", "norm_attn", "norm_mlp")},
                          0, 0)
    # the fp32 path takes the tiny model's odd sizes (d_ff = 688)
    assert B.ax_workspace_bytes(B.make_config(I.SHAPES["tiny"], 1024, 64)) > 0


@pytest.mark.parametrize("name,max_pos,max_tokens,max_seqs,most", [
    ("1b", 8192, 256, 1, 2666.5e6), ("1b", 8192, 1024, 1, 2746.0e6), ("1b", 5000, 4096, 1, 3099.5e6), ("1b", 2048, 64, 4, 2546.5e6),
    ("3b", 8192, 1024, 1, 6780.0e6), ("3b", 8192, 256, 16, 6667.5e6), ("3b", 9000, 3520, 16, 7202.5e6),
    ("8b", 9000, 1024, 1, 15476.5e6), ("8b", 16384, 512, 1, 15349.0e6)])
def test_workspace_stays_the_size_callers_planned_for(name, max_pos, max_tokens, max_seqs, most):
    """Workspace bytes of the decoder shapes.  Attention records: two passes of at most max(2048, one slice) records, which also hold
    every set of items that runs at once (256 compute units x up to 4 blocks x 4 tiles = 4096); a capacity nothing can use once
    made the region four times this size.  The bounds leave 1 MB for descriptors."""
    assert 0 < B.ax_workspace_bytes(B.make_config(I.SHAPES[name], max_pos, max_tokens, max_seqs)) <= most


def test_split_attention_plan():
    """Four wavefronts share out a slice only where slices of eight key steps (two each) make a block for each of the 256 compute
    units - many items over a few steps have nothing to share out; slices of two steps per wavefront at least, a power of
    two, and no more records than a pass has."""
    cfg = B.make_config(I.SHAPES["3b"], 8192, 1024, 64)
    for items in list(range(1, 40)) + [64, 96, 128, 200, 255, 256, 257, 384, 768, 1024, 2000]:
        for steps in list(range(1, 20)) + [24, 31, 32, 41, 64, 137, 256, 273]:
            waves, slices = B.ax_dbg_split_plan(cfg, items, steps)
            assert waves == (4 if items * (steps // 8) >= 256 else 1), (items, steps)
            assert slices & (slices - 1) == 0 and items * slices <= 2048 and (slices == 1 or steps >= 2 * waves * slices), (items, steps, slices)
    assert B.ax_dbg_split_plan(cfg, 384, 3) == (1, 1)
    assert B.ax_dbg_split_plan(cfg, 16, 137)[0] == 4 and B.ax_dbg_split_plan(cfg, 8, 41)[0] == 1
    for items, steps in ((0, 5), (5, 0), (1 << 20, 5)):
        with pytest.raises(B.AxError):
            B.ax_dbg_split_plan(cfg, items, steps)


def test_shared_prefix_plan():
    """Slices of the pass over a shared prefix: none empty, none under two key steps but one, and their records fit a pass's; no more blocks than run
    at once.  Where the pass has the chip to itself (a launch of its own, or little private work beside it) it leaves few compute units without a
    block: 5 groups x 8 heads in 6 slices, not 4; two blocks on a unit for many groups over many keys."""
    for name in ("1b", "3b", "8b"):
        sh = I.SHAPES[name]
        cfg, hd64 = B.make_config(sh, 8192, 1024, 64), sh.head_dim == 64
        for rows in list(range(2, 150)) + [200, 288, 400, 600, 832, 1024]:
            for keys in (32, 64, 96, 160, 1024, 2112, 2496, 6144, 8160):
                tiles, steps = -(-rows // 9), keys // 32
                for own, one in ((2 * tiles, False), (16 * tiles, True), (200 * tiles, True)):
                    groups, slices = B.ax_dbg_shared_plan(cfg, rows, keys, tiles, own, one)
                    blocks = groups * 8
                    assert groups == -(-rows * (sh.n_q_heads // sh.n_kv_heads) // 128)
                    assert slices == 1 or (blocks * slices <= (384 if one and not hd64 else 768) and slices * 2 <= steps), (name, rows, keys, own, one)
                    assert blocks * slices * 4 <= (1024 * (sh.n_q_heads // 8) // 32 + 8 * 64 + 2) * 8
                    assert slices & (slices - 1) == 0 or -(-steps // slices) * (slices - 1) < steps
                    if not hd64 and steps * blocks >= 2 * 256 * 4 and not (one and own * 2 > groups * 4 * steps):
                        assert blocks * slices >= 160, (name, rows, keys, own, one, slices)
    plan = lambda name, *a: B.ax_dbg_shared_plan(B.make_config(I.SHAPES[name], 8192, 1024, 64), *a)
    assert plan("8b", 144, 6144, 32, 96, False) == (5, 6)                     # 16 sessions of 9 rows, short histories
    assert plan("8b", 144, 2496, 32, 1504, True) == (5, 4) and plan("8b", 144, 6144, 32, 1504, True) == (5, 6)
    assert plan("3b", 144, 6144, 16, 48, False) == (4, 8) and plan("3b", 72, 6144, 8, 24, False) == (2, 16)
    assert plan("3b", 288, 6144, 32, 96, False) == (7, 9) and plan("3b", 288, 2496, 32, 96, False) == (7, 4)
    assert plan("8b", 576, 6144, 128, 384, False) == (18, 3) and plan("3b", 360, 6144, 40, 640, True)[1] == 4
    assert plan("1b", 144, 2048, 32, 96, False) == (5, 8)
    for args in ((0, 64, 1, 0), (1025, 64, 1, 0), (9, 31, 1, 0), (9, 64, 0, 0), (9, 64, 1, -1)):
        with pytest.raises(B.AxError):
            plan("3b", *args, False)


def test_attention_merge_plan():
    """A block per record walks the record's slices one after the other, blocks of 4 channels cost their number: the first for many records of few
    slices.  8 sessions over a shared prefix (64 records, 16 shared slices and their own) are the second's, 7.9 us against 11-13."""
    for slices in (17, 18, 20, 24):
        assert not B.ax_dbg_merge_plan(64, slices)
    for records, slices in ((64, 8), (96, 10), (96, 18), (128, 18), (192, 18), (256, 10)):
        assert B.ax_dbg_merge_plan(records, slices), (records, slices)
    for records, slices in ((8, 64), (16, 8), (48, 8), (63, 1), (64, 33), (128, 34), (4096, 33)):
        assert not B.ax_dbg_merge_plan(records, slices), (records, slices)
    for records, slices in ((0, 4), (4, 0)):
        with pytest.raises(B.AxError):
            B.ax_dbg_merge_plan(records, slices)


def test_many_row_gemm_plans_are_launchable():
    """Every plan names a block that is built (block kernel: SwiGLU has no 128 x 128 one; tile kernel: QKV and residual GEMMs of up to 512
    rows; streaming blocks: SwiGLU, up to 192 rows, 128 in hi + lo parts) and K slices that are whole, long enough, and fit
    the scratch and the kernels that add them up."""
    rng = np.random.default_rng(4)
    seen = set()
    for _ in range(6000):
        epi, split = int(rng.integers(0, 4)), bool(rng.integers(0, 2))
        M, N, K = int(np.exp(rng.uniform(np.log(257), np.log(6000)))), 64 * int(rng.integers(1, 260)), 64 * int(rng.integers(1, 260))
        ws = int(rng.choice([0, M * N * 4, 3 * M * N * 4 - 1, 32 * M * N]))
        kernel, rows, cols, slices = B.ax_dbg_gemm_plan(epi, M, N, K, split, ws)
        seen.add((epi, kernel, rows, cols, slices > 1))
        assert slices >= 1 and (slices == 1 or (epi in (1, 3) and slices * M * N * 4 <= ws))
        if kernel == "block":
            assert (rows, cols) in ((256, 256), (128, 256)) + (((128, 128),) if epi != 2 else ())
            assert slices <= 4 and K % (32 * slices) == 0 and (slices == 1 or K // slices >= 512)
        elif kernel == "tile":
            assert epi in (1, 3) and M <= 512 and rows in (64, 128) and cols == 128 and slices <= 8 and K % (64 * slices) == 0
            assert epi == 1 or M * N * 4 <= ws                       # QKV products go through a slab whatever the slices
        else:
            assert kernel == "stream" and epi == 2 and (cols, slices) == (256, 1) and rows in ((96, 128) if split else (96, 128, 160, 192))
    assert len(seen) >= 20, seen
    assert B.ax_dbg_gemm_plan(1, 256, 2048, 2048)[0] == "" == B.ax_dbg_gemm_plan(1, 512, 2064, 2048)[0]


# (epilogue, rows, N, K, hi + lo parts) of decoder layers 2048, 3072 and 4096 wide: choices whose alternatives took 8-50 % longer
@pytest.mark.parametrize("epi,M,N,K,split,want", [
    (3, 288, 3072, 2048, False, ("tile", 64, 128, 2)), (3, 768, 5120, 3072, False, ("block", 128, 128, 1)), (3, 3072, 7168, 5120, False, ("block", 128, 256, 1)),
    (3, 1280, 3072, 2048, False, ("block", 128, 128, 1)), (1, 512, 2048, 8192, False, ("tile", 128, 128, 4)),
    (1, 257, 3072, 8192, False, ("tile", 64, 128, 2)), (1, 768, 3072, 8192, False, ("block", 256, 256, 4)),
    (1, 1280, 3072, 3072, False, ("block", 128, 256, 2)), (1, 640, 4096, 14336, False, ("block", 256, 256, 4)),
    (2, 320, 14336, 4096, False, ("stream", 160, 256, 1)), (2, 576, 14336, 4096, True, ("stream", 96, 256, 1)),
    (2, 4096, 8192, 2048, False, ("block", 256, 256, 1)), (2, 288, 8192, 2048, False, ("block", 128, 256, 1))])
def test_many_row_gemm_plan_of_measured_calls(epi, M, N, K, split, want):
    assert B.ax_dbg_gemm_plan(epi, M, N, K, split, 8 * M * 4096 * 4) == want


def test_strip_gemm_plans_are_launchable():
    """Plans of a layer's GEMMs of 17 to 256 rows: a tile of the register kernel that is built for the epilogue, K slices only of residual GEMMs, long enough and
    within the scratch; blocks, as the block kernel has them, only for hi + lo parts."""
    rng = np.random.default_rng(8)
    seen = set()
    plain = {(2, 1), (2, 2), (2, 4), (3, 2), (3, 3), (3, 4), (4, 2), (4, 3), (4, 4), (5, 4), (6, 4), (8, 4), (9, 4)} | {(m, 8) for m in range(2, 9)}
    for _ in range(6000):
        epi, split = int(rng.integers(1, 4)), bool(rng.integers(0, 2))
        M, N, K = int(rng.integers(17, 257)), 64 * int(rng.integers(1, 260)), 64 * int(rng.integers(1, 260))
        ws = int(rng.choice([0, M * N * 4, 3 * M * N * 4 - 1, 32 * M * N]))
        kernel, rows, cols, slices = B.ax_dbg_strip_plan(epi, M, N, K, split, ws)
        seen.add((epi, kernel, rows, cols, slices > 1))
        assert slices == 1 or slices * M * N * 4 <= ws
        if kernel == "block":
            assert split and (rows, cols) in ((256, 256), (128, 256)) + (((128, 128),) if epi != 2 else ())
            assert slices <= 4 and (slices == 1 or (epi != 2 and K % (32 * slices) == 0 and K // slices >= 512))
        else:
            mt, nt = rows // 16, cols // 16
            assert kernel == "regs" and (mt, nt) in plain - ({(3, 3), (4, 3)} if split else set()) and mt <= -(-M // 16) + 1
            assert (nt >= 2 if slices > 1 else mt <= 5 and nt <= 4) if epi == 1 else nt % 2 == 0 and slices == 1
            assert slices in (1, 2, 4, 8) and (slices == 1 or K // 32 // slices >= 16)
    assert len(seen) >= 60, len(seen)
    for M, N in ((16, 2048), (257, 2048), (64, 2064)):
        with pytest.raises(B.AxError):
            B.ax_dbg_strip_plan(1, M, N, 2048)


# (epilogue, rows, N, K, hi + lo parts) of decoder layers 2048, 3072 and 4096 wide
@pytest.mark.parametrize("epi,M,N,K,split,want", [
    (3, 17, 3072, 2048, False, ("regs", 32, 32, 1)), (2, 64, 8192, 2048, False, ("regs", 64, 64, 1)), (1, 100, 2048, 8192, False, ("regs", 64, 64, 4)),
    (2, 256, 8192, 2048, False, ("regs", 128, 128, 1)), (1, 256, 2048, 8192, False, ("regs", 64, 128, 4)),
    (3, 144, 5120, 3072, False, ("regs", 48, 64, 1)), (1, 144, 3072, 3072, False, ("regs", 48, 48, 1)), (2, 144, 8192, 3072, False, ("regs", 144, 64, 1)),
    (1, 144, 3072, 8192, False, ("regs", 144, 64, 4)), (3, 17, 6144, 4096, True, ("regs", 32, 32, 1)), (2, 17, 14336, 4096, True, ("regs", 32, 128, 1)),
    (3, 112, 6144, 4096, True, ("block", 128, 128, 4)), (2, 160, 14336, 4096, True, ("regs", 80, 128, 1)),
    (2, 224, 14336, 4096, True, ("block", 128, 256, 1)), (1, 224, 4096, 14336, True, ("regs", 112, 128, 4))])
def test_strip_gemm_plan_of_measured_calls(epi, M, N, K, split, want):
    assert B.ax_dbg_strip_plan(epi, M, N, K, split, 8 * M * 4096 * 4) == want


def test_block_gemm_takes_strips_in_hi_and_lo_parts_only():
    """The block kernel has no strips of plain activations (it would read them as panels and write rows): refused on the host, like layouts the
    register kernel does not know.  (The pointers are never followed.)"""
    base = dict(slices=1, M=64, N=192, K=64, A=64, W=64, W2=64, C=64, C16=64, gain=64, ssq_out=64)
    for epi, layouts in ((0, dict(a_panels=2)), (1, dict(a_panels=2)), (1, dict(a_panels=1, c_panels=2)), (2, dict(c_panels=2))):
        with pytest.raises(B.AxError):
            B.ax_dbg_gemm_block(**base, epilogue=epi, rows=128, cols=256, **layouts)
    for layouts in (dict(a_panels=3), dict(a_panels=-1), dict(c_panels=3)):
        with pytest.raises(B.AxError):
            B.ax_dbg_gemm_regs(**base, epilogue=1, rows=32, cols=32, **layouts)


def test_extend_rejects_bad_arguments_before_any_launch():
    cfg = B.make_config(I.SHAPES["tiny"], 1024, 64)
    pool = B.ax_pool_create(cfg, 0, B.ax_pool_block_bytes(cfg) * 8)
    kv = B.ax_kv_alloc(pool)
    for model in (0, 12345):                                   # NULL model handle is refused
        with pytest.raises((B.AxError, OSError, ctypes.ArgumentError)):
            if model == 0:
                B.ax_extend(model, kv, [1, 2, 3])
            else:
                raise B.AxError(B.AX_ERR_INVALID)
    assert B.ax_kv_len(kv) == 0
    B.ax_kv_free(kv)
    B.ax_pool_destroy(pool)


def test_panel_plans_are_launchable():
    """Plans of GEMMs whose activations lie in panels: a block that is built and K slices that are whole, long enough and fit the scratch.
    Calls of up to 16 rows keep panels, those of 17 to 32 unless activations are split, those of 33 to 256 never."""
    rng = np.random.default_rng(7)
    seen = set()
    for _ in range(6000):
        epi, split = int(rng.integers(0, 4)), bool(rng.integers(0, 2))
        M, N, K = int(np.exp(rng.uniform(np.log(257), np.log(6000)))), 64 * int(rng.integers(1, 260)), 64 * int(rng.integers(1, 260))
        ws = int(rng.choice([0, M * N * 4, 3 * M * N * 4 - 1, 32 * M * N]))
        rows, cols, slices = B.ax_dbg_panel_plan(epi, M, N, K, split, ws)
        seen.add((epi, rows, cols, slices > 1))
        assert (rows, cols) in ((256, 256), (128, 256)) + (((128, 128),) if epi != 2 else ())
        assert 1 <= slices <= 4 and (slices == 1 or (epi in (1, 3) and slices * M * N * 4 <= ws and K % (32 * slices) == 0 and K // slices >= 512))
    assert len(seen) >= 14, seen
    for M, N in ((256, 2048), (512, 2064)):
        with pytest.raises(B.AxError):
            B.ax_dbg_panel_plan(1, M, N, 2048)
    for name in ("1b", "3b", "8b"):
        cfg = B.make_config(I.SHAPES[name], 8192, 4096)
        few = name != "8b"                      # (the ~8B shape splits its activations)
        assert [B.ax_dbg_layer_panels(cfg, r) for r in (1, 16, 17, 32, 33, 256, 1024, 4096)] == [True, True, few, few, False, False, True, True]
    assert not B.ax_dbg_layer_panels(B.make_config(I.SHAPES["tiny"], 1024, 64), 9)


@pytest.mark.parametrize("name,rows", [("1b", 288), ("3b", 304), ("8b", 288)])
def test_rows_or_panels_as_measured(name, rows):
    """Whole calls of 257 rows: in rows 1665 / 3834 / 11390 us, in panels 1759 / 3925 / 11780; of 384 rows panels are 1-4 % ahead."""
    cfg = B.make_config(I.SHAPES[name], 8192, 4096)
    assert [B.ax_dbg_layer_panels(cfg, r) for r in (257, rows, 336, 384, 512, 1024)] == [False, False, True, True, True, True]
