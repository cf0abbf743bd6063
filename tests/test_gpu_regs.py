"""GEMMs of 17 to 256 rows: every tile of the register kernel, and the block kernel on strips, against float64."""
import numpy as np
import pytest

from oracle import decoder as O
from paper_2605_10380_amd import inputs as I
from test_gpu_many_rows import BLOCKS, QKV, RESIDUAL, SWIGLU, fp16_bound, operands, panels, rows_of, torch, value  # noqa: F401

pytestmark = pytest.mark.gpu
ROWS, PANELS, STRIPS = 0, 1, 2
TILES = [(2, 1), (2, 2), (2, 4), (3, 2), (3, 3), (3, 4), (4, 2), (4, 3), (4, 4), (5, 4), (6, 4), (8, 4), (9, 4), (2, 8), (3, 8), (4, 8),
         (5, 8), (6, 8), (7, 8), (8, 8)]
HI_LO_TILES = [t for t in TILES if t not in ((3, 3), (4, 3))]
# (epilogue, K slices): QKV and SwiGLU take column tiles in pairs, residual GEMMs finish small tiles on their own
CASES = [(split, epi, slices, mt, nt) for split in (0, 1) for mt, nt in (HI_LO_TILES if split else TILES)
         for epi, slices in ((QKV, 1), (SWIGLU, 1), (RESIDUAL, 1), (RESIDUAL, 2))
         if (nt % 2 == 0 if epi != RESIDUAL else nt >= 2 if slices > 1 else mt <= 5 and nt <= 4)]


def strips(x):
    """[.., M, K] -> [.., ceil16(M) * K]: 32 columns at a time, panels of 16 rows, rows past M any value (NaN here)."""
    *lead, M, K = x.shape
    P = (M + 15) // 16
    full = np.full((*lead, P * 16, K), np.nan, x.dtype)
    full[..., :M, :] = x
    t = full.reshape(*lead, P, 16, K // 32, 4, 8)
    n = len(lead)
    return np.ascontiguousarray(t.transpose(*range(n), n + 2, n, n + 3, n + 1, n + 4)).reshape(*lead, -1)


def unstrips(x, M, K):
    lead, P = x.shape[:-1], (M + 15) // 16
    n = len(lead)
    t = x.reshape(*lead, K // 32, P, 4, 16, 8).transpose(*range(n), n + 1, n + 3, n, n + 2, n + 4)
    return t.reshape(*lead, P * 16, K)[..., :M, :]


@pytest.mark.parametrize("split,epi,slices,mt,nt", CASES)
def test_register_gemm(torch, split, epi, slices, mt, nt):
    """A block of rows and a part of one in strips; whole blocks in rows with fewer chunks of K than wavefronts; a last panel of a few rows in panels.
    Columns end inside a tile (320), K (576) is no whole number of chunks a wavefront.  A pending norm of 5 and of 70 partial sums a row."""
    from paper_2605_10380_amd import binding as B
    check_gemm(torch, B.ax_dbg_gemm_regs, split, epi, slices, 16 * mt, 16 * nt, mt * 100 + nt * 10 + epi + split,
               ((min(mt * 16 + 5, 256), 576, 64, STRIPS, 70), (mt * 16, 64 * slices, 128, ROWS, 5), (max(17, mt * 16 - 11), 320, 64, PANELS, 5)))


@pytest.mark.parametrize("rows,cols,epi,slices", [(r, c, epi, slices) for r, c in BLOCKS for epi in (RESIDUAL, SWIGLU, QKV) for slices in (1, 3)
                                                  if not (epi == SWIGLU and ((r, c) == (128, 128) or slices > 1))])
def test_block_gemm_on_strips(torch, rows, cols, epi, slices):
    """Hi + lo parts in strips on the block kernel, which takes them at 17 to 256 rows where it multiplies faster: a block that is mostly padding,
    a last panel of 1, 4 and 13 rows, whole panels, more rows than a block's 128."""
    from paper_2605_10380_amd import binding as B
    check_gemm(torch, B.ax_dbg_gemm_block, 1, epi, slices, rows, cols, rows + cols + epi, ((20, 192, 64, STRIPS, 70), (109, 576, 128, STRIPS, 5),
                                                                                       (177, 192, 64, STRIPS, 33), (256, 576, 64, STRIPS, 64)))


def check_gemm(torch, gemm, split, epi, slices, tile_rows, tile_cols, seed, calls):
    """Calls of (rows, K, head_dim, layout, partial sums behind the pending norm) on one tile against float64."""
    for M, K, hd, layout, n_sums in calls:
        rng = np.random.default_rng(seed)
        N, Hq = (640 if hd == 128 and epi == QKV else 320), 3
        parts, a, w = operands(rng, M, N, K, split)
        dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()
        bf = lambda x: torch.from_numpy(x).view(torch.bfloat16).cuda()
        lay = {ROWS: lambda x: x, PANELS: panels, STRIPS: strips}[layout]
        rows = (M + 15) // 16 * 16 if layout == STRIPS else M
        by_part = layout == STRIPS or (layout == PANELS and M > 32)
        keep = dict(A=dev(lay(parts)), W=bf(w))
        args = dict(epilogue=epi, rows=tile_rows, cols=tile_cols, slices=slices, M=M, N=N, K=K, a_lo=rows * K if split else 0, a_panels=layout)
        ref = a @ O.widen(w).T
        if epi != RESIDUAL:
            ssq = rng.uniform(0.1, 2.0, (M, n_sums)).astype(np.float32)
            keep["ssq"] = dev(ssq.T if by_part else ssq)
            args.update(n_parts=n_sums, eps=1e-5)
            inv = 1 / np.sqrt(ssq.astype(np.float64).sum(1, keepdims=True) / K + 1e-5)
            ref *= inv
        if slices > 1:
            keep["split_ws"] = torch.full((slices * M * N,), float("nan"), dtype=torch.float32, device="cuda")
            args["split_ws_bytes"] = slices * M * N * 4
        n16 = Hq * hd if epi == QKV else N
        c16 = torch.full((1 + split, (M if epi == QKV else rows) * n16), float("nan"), dtype=torch.float16, device="cuda")
        keep["C16"] = c16
        args["c_lo"] = c16.shape[1] if split else 0
        if epi != QKV:
            args["c_panels"] = layout
        unlay = lambda t: t.reshape(1 + split, M, n16) if layout == ROWS or epi == QKV else rows_of(t, M, n16) if layout == PANELS else unstrips(t, M, n16)
        got16 = lambda: value(torch.from_numpy(np.ascontiguousarray(unlay(c16.cpu().numpy()))), split)
        if epi == RESIDUAL:
            c0, gain = rng.standard_normal((M, N), dtype=np.float32), I.f32_to_bf16_bits(1.0 + 0.1 * rng.standard_normal(N, dtype=np.float32))
            keep.update(C=dev(c0.copy()), gain=bf(gain), ssq_out=torch.full((M * N // 8,), float("nan"), dtype=torch.float32, device="cuda"))
        if epi == SWIGLU:
            w2 = I.f32_to_bf16_bits(rng.standard_normal((N, K), dtype=np.float32) * 0.05)
            keep["W2"] = bf(w2)
        if epi == QKV:
            Hkv, n_blocks = (N // hd - Hq) // 2, 40
            pos, slot = rng.integers(0, 500, M).astype(np.int32), rng.permutation(n_blocks * 16)[:M].astype(np.int32)
            ang = np.arange(500)[:, None] * 10000.0 ** (-2.0 * np.arange(hd // 2) / hd)
            pool = torch.full((2, Hkv, n_blocks, 16 * hd), float("nan"), dtype=torch.float16, device="cuda")
            keep.update(pool=pool, row_pos=dev(pos), row_slot=dev(slot), cos=dev(np.cos(ang).astype(np.float32)), sin=dev(np.sin(ang).astype(np.float32)))
            args.update(n_q_heads=Hq, n_kv_heads=Hkv, head_dim=hd, pool_blocks=n_blocks)
        torch.cuda.synchronize()
        n_out = gemm(**args, **{k: t.data_ptr() for k, t in keep.items()})
        what = (M, K, layout)
        if epi == RESIDUAL:
            want, got = c0 + ref, keep["C"].cpu().numpy().astype(np.float64)
            assert np.abs(got - want).max() <= 2e-5 * np.abs(want).max(), what
            want16 = got * O.widen(gain)[None, :]
            assert (np.abs(got16() - want16) <= fp16_bound(want16, split)).all(), what
            sums = keep["ssq_out"].cpu().numpy()[:M * n_out]
            sums = (sums.reshape(n_out, M).T if by_part else sums.reshape(M, n_out)).astype(np.float64).sum(1)
            assert np.allclose(sums, (want ** 2).sum(1), rtol=4e-5), what
        elif epi == SWIGLU:
            up = a @ O.widen(w2).T * inv
            want = O.silu(ref) * up
            # gate and up: 2e-5 of their largest values each, and __expf's few units in the last place of fp32
            assert (np.abs(got16() - want) <= fp16_bound(want, split) + 4e-5 * np.abs(ref).max() * np.abs(up).max()).all(), what
        else:
            qkv = ref.reshape(M, -1, hd)
            half, cs, sn = hd // 2, np.cos(ang[pos])[:, None], np.sin(ang[pos])[:, None]
            rot = lambda t: np.concatenate([t[..., :half] * cs - t[..., half:] * sn, t[..., half:] * cs + t[..., :half] * sn], -1)
            wq, wk, wv = rot(qkv[:, :Hq]), rot(qkv[:, Hq:Hq + Hkv]), qkv[:, Hq + Hkv:]
            assert (np.abs(got16().reshape(M, Hq, hd) - wq) <= fp16_bound(wq, split)).all(), what
            mem = pool.cpu().numpy().astype(np.float64)
            k = mem[0].reshape(Hkv, n_blocks * 16, hd)
            v = mem[1].reshape(Hkv, n_blocks, hd, 16).transpose(0, 1, 3, 2).reshape(Hkv, n_blocks * 16, hd)
            assert (np.abs(k[:, slot] - wk.transpose(1, 0, 2)) <= fp16_bound(wk, 0).transpose(1, 0, 2)).all(), what
            assert (np.abs(v[:, slot] - wv.transpose(1, 0, 2)) <= fp16_bound(wv, 0).transpose(1, 0, 2)).all(), what
            rest = np.setdiff1d(np.arange(n_blocks * 16), slot)                  # no slot but the rows' own was written
            assert np.isnan(k[:, rest]).all() and np.isnan(v[:, rest]).all(), what


def test_tiles_that_are_not_built_are_refused(torch):
    from paper_2605_10380_amd import binding as B
    t = torch.zeros(1 << 16, device="cuda")
    p = t.data_ptr()
    for args in (dict(epilogue=QKV, rows=48, cols=48), dict(epilogue=RESIDUAL, rows=128, cols=128), dict(epilogue=0, rows=32, cols=32),
                 dict(epilogue=SWIGLU, rows=32, cols=32, slices=2), dict(epilogue=SWIGLU, rows=64, cols=32, M=257)):
        with pytest.raises(B.AxError):
            B.ax_dbg_gemm_regs(**dict(dict(slices=1, M=32, N=192, K=64, A=p, W=p, W2=p, C=p, C16=p, gain=p, ssq_out=p, split_ws=p, split_ws_bytes=1 << 17,
                                           n_q_heads=1, n_kv_heads=1, head_dim=64, pool=p, pool_blocks=1, row_pos=p, row_slot=p, cos=p, sin=p), **args))


# one layer, hi + lo parts or not, and what its plans take for QKV, O, gate / up and down (with K slices): the register kernel whole and in slices; hi + lo
# parts with gate / up, QKV in slices and both residual GEMMs on blocks
LAYERS = [((256, 4, 2, 64, 320), 40, 0, ("regs", "regs", "regs", "regs")), ((512, 8, 2, 64, 8192), 48, 0, ("regs", "regs", "regs", "regs4")),
          ((1024, 8, 4, 128, 9216), 201, 1, ("regs", "regs", "block", "regs8")), ((4096, 32, 8, 128, 320), 121, 1, ("block4", "regs4", "regs", "regs")),
          ((9536, 4, 2, 64, 768), 249, 1, ("regs", "block", "regs", "block"))]


@pytest.mark.parametrize("dims,rows,split,plan", LAYERS)
def test_layer_of_17_to_256_rows(torch, dims, rows, split, plan):
    from test_gpu_kernels import _one_layer
    from paper_2605_10380_amd import binding as B
    d, hq, hkv, hd, F = dims
    qkv = (hq + 2 * hkv) * hd
    got = [B.ax_dbg_strip_plan(e, rows, n, k, bool(split), 256 * max(8 * d, qkv) * 4) for e, n, k in ((QKV, qkv, d), (RESIDUAL, d, hq * hd), (SWIGLU, F, d), (RESIDUAL, d, F))]
    assert tuple(k + (str(s) if s > 1 else "") for k, _, _, s in got) == plan
    sh = I.DecoderShape("strips", 1, d, hq, hkv, hd, F, 512, "bf16")
    attn, attn_ref, x, x_ref = _one_layer(torch, sh, 37, rows, 24, 256, split)
    assert np.abs(attn - attn_ref).max() <= 4e-3 * np.abs(attn_ref).max()
    assert np.abs(x - x_ref).max() <= 4e-3 * np.abs(x_ref).max()
