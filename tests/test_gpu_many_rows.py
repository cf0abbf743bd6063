"""GPU: the kernels behind calls of more than 256 rows, every tile shape x epilogue x slicing x activation layout against float64, and
the calls whose plan picks them."""
import numpy as np
import pytest

from oracle import decoder as O
from paper_2605_10380_amd import inputs as I

pytestmark = pytest.mark.gpu

BLOCKS = [(256, 256), (128, 256), (128, 128)]
STORE, RESIDUAL, SWIGLU, QKV = range(4)


@pytest.fixture(scope="module")
def torch():
    import torch
    assert torch.cuda.is_available()
    return torch


def hi_lo(x):
    """[2, ...]: fp16 hi and lo parts."""
    hi = x.astype(np.float16)
    return np.stack([hi, (x - hi.astype(np.float64)).astype(np.float16)])


def operands(rng, M, N, K, split):
    a = rng.standard_normal((M, K)) * 0.5
    parts = hi_lo(a) if split else a.astype(np.float16)[None]
    w = I.f32_to_bf16_bits(rng.standard_normal((N, K), dtype=np.float32) * 0.05)
    return parts, parts.astype(np.float64).sum(0), w


def value(t, split):
    """Value of a result that came as hi + lo parts, or as fp16."""
    x = t.cpu().numpy().astype(np.float64)
    return x[0] + x[1] if split else x[0]


def fp16_bound(want, split):
    """fp16: 2^-11 of the value; hi + lo parts: 2^-22, and what is below fp16's smallest subnormal.  Plus fp32 sums as in the other GEMM
    tests: 2e-5 of the largest value."""
    scale = np.abs(want).max()
    return (2.0 ** -22 if split else 2.0 ** -11) * np.abs(want) + 2e-5 * scale + 2.0 ** -24


CASES = [(b, epi, split, slices, hd, K)
         for b in BLOCKS for epi in (STORE, RESIDUAL, SWIGLU, QKV) for split in (0, 1)
         for slices, K in ((1, 64), (1, 576), (3, 576)) for hd in ((64, 128) if epi == QKV else (0,))
         if not (epi == SWIGLU and b == (128, 128)) and not (slices > 1 and epi in (STORE, SWIGLU))]


@pytest.mark.parametrize("block,epi,split,slices,hd,K", CASES)
def test_block_gemm(torch, block, epi, split, slices, hd, K):
    """300 rows (a whole tile and a part of one), columns that end inside a tile, fewer and more steps than stages, whole and in slices, A as
    it is or with a pending norm."""
    from paper_2605_10380_amd import binding as B
    M = 300
    Hq, Hkv = 3, 1
    N = {64: 320, 128: 640}.get(hd, 320)
    rng = np.random.default_rng(hash((block, epi, split, slices, hd, K)) % (1 << 31))
    parts, a, w = operands(rng, M, N, K, split)
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()
    bf = lambda x: torch.from_numpy(x).view(torch.bfloat16).cuda()
    keep = dict(A=dev(parts), W=bf(w))
    args = dict(epilogue=epi, rows=block[0], cols=block[1], slices=slices, M=M, N=N, K=K, a_lo=M * K if split else 0)
    ref = a @ O.widen(w).T
    if epi != RESIDUAL:                                        # the pending norm of A: five partial sums a row
        ssq = rng.uniform(0.1, 2.0, (M, 5)).astype(np.float32)
        keep["ssq"] = dev(ssq)
        args.update(n_parts=5, eps=1e-5)
        ref /= np.sqrt(ssq.astype(np.float64).sum(1, keepdims=True) / K + 1e-5)
    if slices > 1:
        keep["split_ws"] = torch.full((slices * M * N,), float("nan"), dtype=torch.float32, device="cuda")
        args["split_ws_bytes"] = slices * M * N * 4
    n16 = 3 * hd if epi == QKV else N
    c16 = torch.full((1 + split, M, n16), float("nan"), dtype=torch.float16, device="cuda")
    if epi != STORE:
        keep["C16"] = c16
        args["c_lo"] = M * n16 if split else 0
    if epi in (STORE, RESIDUAL):
        c0 = rng.standard_normal((M, N), dtype=np.float32)
        keep["C"] = dev(c0.copy())
    if epi == RESIDUAL:
        gain = I.f32_to_bf16_bits(1.0 + 0.1 * rng.standard_normal(N, dtype=np.float32))
        keep.update(gain=bf(gain), ssq_out=torch.full((M * N // 8,), float("nan"), dtype=torch.float32, device="cuda"))
    if epi == SWIGLU:
        w2 = I.f32_to_bf16_bits(rng.standard_normal((N, K), dtype=np.float32) * 0.05)
        keep["W2"] = bf(w2)
    if epi == QKV:
        Hkv = (N // hd - 3) // 2
        n_blocks = 40
        pos = rng.integers(0, 500, M).astype(np.int32)
        slot = rng.permutation(n_blocks * 16)[:M].astype(np.int32)
        ang = np.arange(500)[:, None] * 10000.0 ** (-2.0 * np.arange(hd // 2) / hd)
        pool = torch.full((2, Hkv, n_blocks, 16 * hd), float("nan"), dtype=torch.float16, device="cuda")
        keep.update(pool=pool, row_pos=dev(pos), row_slot=dev(slot), cos=dev(np.cos(ang).astype(np.float32)), sin=dev(np.sin(ang).astype(np.float32)))
        args.update(n_q_heads=3, n_kv_heads=Hkv, head_dim=hd, pool_blocks=n_blocks)
    torch.cuda.synchronize()
    n_out = B.ax_dbg_gemm_block(**args, **{k: t.data_ptr() for k, t in keep.items()})

    if epi == STORE:
        assert (np.abs(keep["C"].cpu().numpy() - ref) <= 2e-5 * np.abs(ref).max()).all()
    elif epi == RESIDUAL:
        want = c0 + ref
        got = keep["C"].cpu().numpy().astype(np.float64)
        assert np.abs(got - want).max() <= 2e-5 * np.abs(want).max()
        want16 = got * O.widen(gain)[None, :]
        assert (np.abs(value(c16, split) - want16) <= fp16_bound(want16, split)).all()
        assert n_out == (1 if slices > 1 else N // 64)
        sums = keep["ssq_out"].cpu().numpy()[:M * n_out].reshape(M, n_out).astype(np.float64).sum(1)
        assert np.allclose(sums, (want ** 2).sum(1), rtol=4e-5)
    elif epi == SWIGLU:
        up = a @ O.widen(w2).T / np.sqrt(ssq.astype(np.float64).sum(1, keepdims=True) / K + 1e-5)
        want = O.silu(ref) * up
        # gate and up: 2e-5 of their largest values each, and __expf's few units in the last place of fp32
        bound = fp16_bound(want, split) + 4e-5 * np.abs(ref).max() * np.abs(up).max()
        assert (np.abs(value(c16, split) - want) <= bound).all()
    else:
        qkv = ref.reshape(M, -1, hd)
        half, cs, sn = hd // 2, np.cos(ang[pos])[:, None], np.sin(ang[pos])[:, None]
        rot = lambda t: np.concatenate([t[..., :half] * cs - t[..., half:] * sn, t[..., half:] * cs + t[..., :half] * sn], -1)
        wq, wk, wv = rot(qkv[:, :3]), rot(qkv[:, 3:3 + Hkv]), qkv[:, 3 + Hkv:]
        assert (np.abs(value(c16, split).reshape(M, 3, hd) - wq) <= fp16_bound(wq, split)).all()
        mem = pool.cpu().numpy().astype(np.float64)
        k = mem[0].reshape(Hkv, n_blocks * 16, hd)
        v = mem[1].reshape(Hkv, n_blocks, hd, 16).transpose(0, 1, 3, 2).reshape(Hkv, n_blocks * 16, hd)
        assert (np.abs(k[:, slot] - wk.transpose(1, 0, 2)) <= fp16_bound(wk, 0).transpose(1, 0, 2)).all()
        assert (np.abs(v[:, slot] - wv.transpose(1, 0, 2)) <= fp16_bound(wv, 0).transpose(1, 0, 2)).all()
        rest = np.setdiff1d(np.arange(n_blocks * 16), slot)    # no slot but the rows' own was written
        assert np.isnan(k[:, rest]).all() and np.isnan(v[:, rest]).all()
    assert torch.isfinite(c16).all() or epi == STORE


# what the plan picks, and a call that reaches it: (epilogue, M, N, K, plan); few-column cases of every tile, slice count and kernel
PLANNED = [
    (RESIDUAL, 300, 320, 64, ("tile", 64, 128, 1)), (RESIDUAL, 321, 320, 1024, ("tile", 64, 128, 2)), (RESIDUAL, 257, 320, 4096, ("tile", 64, 128, 8)),
    (RESIDUAL, 500, 3136, 4096, ("tile", 128, 128, 2)), (RESIDUAL, 500, 1600, 8192, ("tile", 128, 128, 4)),
    (RESIDUAL, 513, 320, 64, ("block", 128, 128, 1)), (RESIDUAL, 513, 320, 2048, ("block", 128, 128, 4)),
    (RESIDUAL, 513, 3840, 2048, ("block", 128, 256, 2)), (RESIDUAL, 513, 14400, 64, ("block", 128, 256, 1)),      # (285 blocks: two on a compute unit)
    (RESIDUAL, 500, 4160, 4096, ("block", 256, 256, 4)),
    (SWIGLU, 257, 320, 64, ("block", 128, 256, 1)), (SWIGLU, 321, 11072, 512, ("block", 256, 256, 1)),
    (SWIGLU, 500, 320, 3072, ("stream", 96, 256, 1)), (SWIGLU, 257, 14400, 1024, ("stream", 160, 256, 1)),
    (SWIGLU, 513, 10240, 3072, ("stream", 192, 256, 1)),
    # few columns, short K, ragged rows on the blocks
    (RESIDUAL, 257, 320, 64, ("block", 128, 128, 1)), (RESIDUAL, 257, 320, 1024, ("block", 128, 128, 2)),
    (RESIDUAL, 449, 4160, 64, ("block", 128, 128, 1)), (RESIDUAL, 449, 4160, 1024, ("block", 128, 128, 1)),
    (SWIGLU, 385, 14400, 64, ("block", 128, 256, 1)), (SWIGLU, 500, 320, 1024, ("block", 128, 256, 1)),
    (SWIGLU, 257, 14400, 64, ("block", 128, 256, 1)), (SWIGLU, 321, 14400, 64, ("block", 128, 256, 1))]


@pytest.mark.parametrize("epi,M,N,K,plan", PLANNED)
def test_planned_gemm(torch, epi, M, N, K, plan):
    """A GEMM of more than 256 rows on each kernel the plan knows, against float64."""
    import test_gpu_kernels as T
    from paper_2605_10380_amd import binding as B
    assert B.ax_dbg_gemm_plan(epi, M, N, K, False, 8 * M * N * 4) == plan
    if epi == RESIDUAL:
        T.test_bf16_residual_gemm_with_norm_preparation(torch, M, N, K, True)
    else:
        T.test_bf16_gemm(torch, M, N, K, epi)


@pytest.mark.parametrize("M,N,K,split", [(1600, 7744, 192, True), (1030, 5056, 8192, True), (1664, 7680, 448, True)])
def test_residual_gemm_of_many_rows(torch, M, N, K, split):
    """The residual epilogue with norm preparation over a thousand rows, columns that are no multiple of a tile."""
    import test_gpu_kernels as T
    T.test_bf16_residual_gemm_with_norm_preparation(torch, M, N, K, split)


def _random_many_row_cases(n=18, seed=20260519):
    """Seeded shapes above 256 rows with N a multiple of 64, as every model's are: all epilogues of the debug entry."""
    rng = np.random.default_rng(seed)
    return [(int(np.exp(rng.uniform(np.log(257), np.log(1700)))), 64 * int(rng.integers(1, 100)), 64 * int(rng.integers(1, 40)), i % 3) for i in range(n)]


@pytest.mark.parametrize("M,N,K,epi", _random_many_row_cases())
def test_many_row_gemm_seeded_random_shapes(torch, M, N, K, epi):
    import test_gpu_kernels as T
    T.test_bf16_gemm(torch, M, N, K, epi)


# one layer, hi + lo activations or not, and the kernels of its four GEMMs (QKV, O, gate / up, down): layers that keep rows, and layers in panels
LAYERS = [
    ((256, 4, 2, 64, 320, 300, 0), ("block", "tile", "block", "tile")),
    ((384, 4, 2, 64, 2816, 257, 1), ("tile", "block", "block", "tile")), ((384, 8, 2, 64, 2816, 257, 1), ("tile", "tile", "block", "tile")),
    ((704, 4, 2, 64, 14336, 320, 0), ("block", "tile", "stream", "tile")), ((2048, 16, 4, 128, 1088, 257, 1), ("tile", "block", "block", "block")),
    ((2048, 4, 2, 64, 10240, 270, 1), ("block", "tile", "stream", "block"))]
PANEL_LAYERS = [
    ((256, 4, 2, 64, 320, 310, 0), ((128, 128, 1), (128, 128, 1), (128, 256, 1), (128, 128, 1))),
    ((2048, 4, 2, 64, 320, 640, 1), ((128, 128, 4), (128, 128, 1), (128, 256, 1), (128, 128, 1))),
    ((1024, 8, 4, 64, 320, 500, 0), ((128, 128, 2), (128, 128, 1), (128, 256, 1), (128, 128, 1)))]


@pytest.mark.parametrize("dims,plans", LAYERS + PANEL_LAYERS)
def test_layer_of_planned_gemms(torch, dims, plans):
    import test_gpu_kernels as T
    from paper_2605_10380_amd import binding as B
    d, hq, hkv, hd, F, rows, split = dims
    qkv, in_panels = (hq + 2 * hkv) * hd, not isinstance(plans[0], str)
    ws = rows * max(8 * d, qkv) * 4
    sh = I.DecoderShape("planned", 1, d, hq, hkv, hd, F, 512, "bf16")
    assert B.ax_dbg_layer_panels(B.make_config(sh, rows + 16, rows, 1, split), rows) == in_panels
    gemms = ((QKV, qkv, d), (RESIDUAL, d, hq * hd), (SWIGLU, F, d), (RESIDUAL, d, F))
    plan = B.ax_dbg_panel_plan if in_panels else lambda *a: B.ax_dbg_gemm_plan(*a)[0]
    assert tuple(plan(e, rows, n, k, bool(split), ws) for e, n, k in gemms) == plans
    attn, attn_ref, x, x_ref = T._one_layer(torch, sh, 0, rows, 24, rows, split)
    assert np.abs(attn - attn_ref).max() <= 4e-3 * np.abs(attn_ref).max()
    assert np.abs(x - x_ref).max() <= 4e-3 * np.abs(x_ref).max()


@pytest.mark.parametrize("hd,hkv,G,P,T,split,least", [
    (64, 32, 4, 1100, 1056, 0, 1),                             # 33 groups for 32 places a head: the last one is cut
    (64, 2, 4, 4000, 96, 0, 1), (128, 8, 3, 1500, 200, 1, 1)])
def test_block_attention_cut_groups(torch, hd, hkv, G, P, T, split, least):
    """Attention items of groups that are cut beside (first case) groups that write their output themselves."""
    import test_gpu_kernels as K
    from paper_2605_10380_amd import binding as B
    sh = I.DecoderShape("attn-cut", 1, 128, hkv * G, hkv, hd, 192, 512, "bf16")
    items, merges, slots = B.ax_dbg_attention_items(B.make_config(sh, P + T + 16, max(T, 64), 1, split), [P], [T])
    groups = -(-T * G // 128)
    assert merges >= least and items == groups - merges + slots
    if groups > 32:
        assert merges < groups
    got, ref, x, xr = K._one_layer(torch, sh, P, T, 25, max(T, 64), split)
    assert np.abs(got - ref).max() <= 4e-3 * np.abs(ref).max()
    assert np.abs(x - xr).max() <= 4e-3 * np.abs(xr).max()


@pytest.mark.parametrize("d,hq,hkv,hd,F", [(2048, 8, 2, 64, 2048), (1024, 8, 4, 128, 9216)])
@pytest.mark.parametrize("T,calls", [(9, 8), (17, 5), (48, 3), (144, 2), (200, 1), (300, 1), (700, 1)])
def test_hi_and_lo_parts_add_up(torch, d, hq, hkv, hd, F, T, calls):
    """Split activations: hi + lo of the LM head's input is x * gain to 2^-22 whichever kernel finished the residual stream - also where
    x * gain lies so close to a tie that rounding it once or through fp32 makes a difference."""
    from paper_2605_10380_amd import binding as B
    sh = I.DecoderShape("parts", 1, d, hq, hkv, hd, F, 512, "bf16")
    w = I.make_weights(sh, 31)
    gain = O.widen(w["final_norm"])
    dm = B.DeviceModel(sh, w, max_pos=1024, max_tokens=max(T, 64), pool_tokens=1024, act_split=1)
    kv = dm.new_kv()
    rng = np.random.default_rng(T + d)
    for _ in range(calls):
        B.ax_kv_truncate(kv, 0)
        dm.extend(kv, rng.integers(0, sh.vocab, T).astype(np.int32), B.AX_OUT_LAST_ARGMAX)
        x, hi, lo = np.zeros((T, d), np.float32), np.zeros((T, d), np.float16), np.zeros((T, d), np.float16)
        B.ax_dbg_read(dm.model, 0, x)
        B.ax_dbg_read(dm.model, 5, hi)
        B.ax_dbg_read(dm.model, 15, lo)
        want = x.astype(np.float64) * gain
        # fp32 product 2^-24, lo part 2^-11 of half an fp16 step, and lo parts below the smallest subnormal
        err = np.abs(hi.astype(np.float64) + lo.astype(np.float64) - want)
        assert (err <= 2.0 ** -22 * np.abs(want) + 2.0 ** -24).all(), (int((err > 2.0 ** -22 * np.abs(want) + 2.0 ** -24).sum()), err.max())
    B.ax_kv_free(kv)
    dm.close()


def panels(x):
    """[.., M, K] -> [.., M * K], 16-row panels: a panel's rows of 8 columns at a time, a short last panel in shorter runs."""
    *lead, M, K = x.shape
    return np.concatenate([x[..., r:r + 16, :].reshape(*lead, -1, K // 8, 8).swapaxes(-3, -2).reshape(*lead, -1) for r in range(0, M, 16)], -1)


def rows_of(x, M, K):
    """The inverse of panels."""
    out = np.empty((*x.shape[:-1], M, K), x.dtype)
    for r in range(0, M, 16):
        n = min(16, M - r)
        out[..., r:r + n, :] = x[..., r * K:(r + n) * K].reshape(*x.shape[:-1], K // 8, n, 8).swapaxes(-3, -2).reshape(*x.shape[:-1], n, K)
    return out


PANEL_CASES = [(b, epi, split, slices, M, N, K, parts, 64)
               for b in BLOCKS for epi in (STORE, RESIDUAL, SWIGLU, QKV) for split in (0, 1)
               for slices, M, N, K, parts in ((1, 300, 320, 576, 5), (1, 257, 640, 64, 33), (3, 385, 320, 576, 64))
               if not (epi == SWIGLU and b == (128, 128)) and not (slices > 1 and epi in (STORE, SWIGLU))]
PANEL_CASES += [(b, QKV, split, slices, M, 640, 576, parts, 128) for b in BLOCKS for split in (0, 1) for slices, M, parts in ((1, 300, 64), (3, 270, 33))]
# more than 256 blocks of 128 x 256: two on a compute unit
PANEL_CASES += [((128, 256), epi, 0, 1, 300, 22080 if epi != SWIGLU else 11072, K, 1, 64) for epi in (STORE, RESIDUAL, SWIGLU, QKV) for K in (64, 160 * 2)]
PANEL_CASES += [((128, 256), RESIDUAL, 0, 3, 300, 7424, 576, 1, 64)]


@pytest.mark.parametrize("block,epi,split,slices,M,N,K,n_sums,hd", PANEL_CASES)
def test_block_gemm_in_panels(torch, block, epi, split, slices, M, N, K, n_sums, hd):
    """Activations in panels, a short last one among them: the same bits as in rows on 256 x 256 blocks (every output is the same sum in the
    same order whatever the block), which the test above holds against float64.  The partial sums of x^2 behind a pending norm, [part][row]
    beside panels and [row][part] beside rows, are multiples of 2^-10 below 2: exact in fp32 in any order."""
    from paper_2605_10380_amd import binding as B
    rng = np.random.default_rng(M + N + K + split)
    parts, _, w = operands(rng, M, N, K, split)
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()
    bf = lambda x: torch.from_numpy(x).view(torch.bfloat16).cuda()
    n16 = N - 2 * hd if epi == QKV else N
    pos, slot = rng.integers(0, 500, M).astype(np.int32), rng.permutation(40 * 16)[:M].astype(np.int32)
    ang = np.arange(500)[:, None] * 10000.0 ** (-2.0 * np.arange(hd // 2) / hd)
    c0, gain = rng.standard_normal((M, N), dtype=np.float32), I.f32_to_bf16_bits(1.0 + 0.1 * rng.standard_normal(N, dtype=np.float32))
    ssq, w2 = (rng.integers(100, 2048, (M, n_sums)) / 1024).astype(np.float32), rng.permutation(w)

    def run(block, in_panels):
        keep = dict(A=dev(panels(parts) if in_panels else parts), W=bf(w))
        args = dict(epilogue=epi, rows=block[0], cols=block[1], slices=slices, M=M, N=N, K=K, a_lo=M * K if split else 0, a_panels=in_panels)
        if epi != RESIDUAL:
            keep["ssq"] = dev(ssq.T if in_panels else ssq)
            args.update(n_parts=n_sums, eps=1e-5)
        if slices > 1:
            keep["split_ws"] = torch.full((slices * M * N,), float("nan"), dtype=torch.float32, device="cuda")
            args["split_ws_bytes"] = slices * M * N * 4
        if epi != STORE:
            keep["C16"] = torch.full((1 + split, M * n16), float("nan"), dtype=torch.float16, device="cuda")
            args["c_lo"] = M * n16 if split else 0
        if epi in (STORE, RESIDUAL):
            keep["C"] = dev(c0.copy())
        if epi in (RESIDUAL, SWIGLU):
            args["c_panels"] = in_panels
        if epi == RESIDUAL:
            keep.update(gain=bf(gain), ssq_out=torch.full((M * N // 8,), float("nan"), dtype=torch.float32, device="cuda"))
        if epi == SWIGLU:
            keep["W2"] = bf(w2)
        if epi == QKV:
            keep.update(pool=torch.full((2, 1, 40, 16 * hd), -7.0, dtype=torch.float16, device="cuda"), row_pos=dev(pos), row_slot=dev(slot),
                        cos=dev(np.cos(ang).astype(np.float32)), sin=dev(np.sin(ang).astype(np.float32)))
            args.update(n_q_heads=N // hd - 2, n_kv_heads=1, head_dim=hd, pool_blocks=40)
        torch.cuda.synchronize()
        n_out = B.ax_dbg_gemm_block(**args, **{k: t.data_ptr() for k, t in keep.items()})
        out = {k: keep[k].cpu().numpy() for k in ("C", "C16", "pool") if k in keep}
        if epi in (RESIDUAL, SWIGLU) and in_panels:
            out["C16"] = rows_of(out["C16"], M, N).reshape(1 + split, -1)
        sums = None
        if epi == RESIDUAL:
            sums = keep["ssq_out"].cpu().numpy()[:M * n_out]
            sums = (sums.reshape(n_out, M).T if in_panels else sums.reshape(M, n_out)).astype(np.float64).sum(1)
        return out, sums

    want, want_sums = run((256, 256), 0)
    for in_panels in (1, 0) if N > 7000 else (1,):             # (two on a compute unit: the same block in rows as well)
        got, sums = run(block, in_panels)
        assert want.keys() == got.keys()
        for k in want:
            assert np.array_equal(want[k], got[k]), (k, in_panels, np.abs(want[k].astype(np.float64) - got[k]).max())
        if epi == RESIDUAL:
            assert np.allclose(sums, want_sums, rtol=1e-5)     # fp32 sums of x^2 in another order


@pytest.mark.parametrize("split", [0, 1])
@pytest.mark.parametrize("T", [1, 2, 7, 8, 9, 15, 16, 17, 18, 24, 31, 32, 33])
@pytest.mark.parametrize("hd,hkv,G,d,F", [(64, 2, 4, 256, 320), (128, 1, 8, 1024, 1600)])
def test_layer_of_one_or_two_panels(torch, hd, hkv, G, d, F, T, split):
    """Calls of up to 16 rows keep their activations in one panel of as many rows, on few-row blocks of 8 and 16 columns; plain ones of up to 32 in
    two, others in strips (33: all in strips), on the register kernel."""
    import test_gpu_kernels as K
    sh = I.DecoderShape("one-panel", 1, d, hkv * G, hkv, hd, F, 512, "bf16")
    got, ref, x, xr = K._one_layer(torch, sh, 37, T, 30 + T, 64, split)
    assert np.abs(got - ref).max() <= 4e-3 * np.abs(ref).max()
    assert np.abs(x - xr).max() <= 4e-3 * np.abs(xr).max()


@pytest.mark.parametrize("T", [5, 300])
def test_embedding_that_is_not_16_byte_aligned(torch, T):
    """The embedding and the gains are read where the caller has them, at any address a bf16 can have."""
    from paper_2605_10380_amd import binding as B
    sh = I.DecoderShape("odd", 1, 128, 2, 1, 64, 192, 512, "bf16")
    w = I.make_weights(sh, 5)
    toks = np.random.default_rng(T).integers(0, sh.vocab, T).astype(np.int32)

    def logits(shift):
        t = {k: [torch.from_numpy(a).view(torch.bfloat16).cuda() for a in v] if isinstance(v, list) else torch.from_numpy(v).view(torch.bfloat16).cuda() for k, v in w.items()}

        def moved(x):
            flat = torch.zeros(x.numel() + 8, dtype=x.dtype, device="cuda")[shift:shift + x.numel()]
            return flat.copy_(x.flatten()).view(x.shape)
        t["tok_emb"], t["norm_attn"] = moved(t["tok_emb"]), [moved(x) for x in t["norm_attn"]]
        dm = B.DeviceModel(sh, t, max_pos=512, max_tokens=T, pool_tokens=512)
        out = dm.extend(dm.new_kv(), toks, B.AX_OUT_ALL_LOGITS).cpu().numpy()
        return out

    assert np.array_equal(logits(0), logits(1)) and np.array_equal(logits(0), logits(3))
