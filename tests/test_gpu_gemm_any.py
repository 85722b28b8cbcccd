"""sbp_matmul on sizes that fit no tile and no reduction step: every remainder of the reduction length, ragged rows and
columns, all four storage layouts, against the oracle.  Padding holds NaN (sbp_harness), so a value read past the end of
a row shows in the result.  Bars: fp32 results differ from the oracle by summation order only, at most
sqrt(K) 2^-24 of the result's scale and far below 1e-5; bf16 results by one rounding, 2^-8 of the value."""
import numpy as np
import pytest

import oracle as orc
import paper_2110_15032_amd as sbp
import workloads as wl
from sbp_harness import DevTensor, TO_ABI, assert_matmul_close, sync, values

pytestmark = pytest.mark.gpu
SEED = wl.SEED_BASE + 1700


def bf16(tid, shape, scale=1.0):
    return wl.to_bf16_bits(wl.normal(SEED, tid, shape, scale))


def pitch(shards, trans, to, extra=0):
    """row pitch: the longest stored row rounded up to a multiple of `to`, plus `extra`"""
    n = max((s.shape[0] if trans else s.shape[1]) for s in shards)
    return -(-n // to) * to + extra


def run(Xs, sx, Ws, sw, M, K, N, k, tx, tw, ldx, ldw, ldy=0, variant=0, epilogue=sbp.EPI_NONE):
    sy = orc.infer_matmul(sx, sw)
    bf = Xs[0].dtype == np.uint16 and Ws[0].dtype == np.uint16
    out_dt = np.uint16 if bf and sy != orc.P_SUM else np.float32
    dx = DevTensor.from_host(Xs, M, K, sx, trans=tx, ld=ldx)
    dw = DevTensor.from_host(Ws, K, N, sw, trans=tw, ld=ldw)
    dy = DevTensor.empty(M, N, out_dt, sy, k, ld=ldy)
    sbp.sbp_set_knob(sbp.KNOB_GEMM_VARIANT, variant)
    try:
        sbp.sbp_matmul_ex(dx.desc, TO_ABI[sx], dw.desc, TO_ABI[sw], dy.desc, sbp.AUTO, k, None, epilogue)
        sync()
    finally:
        sbp.sbp_set_knob(sbp.KNOB_GEMM_VARIANT, 0)
    return [values(y) if out_dt == np.uint16 else y for y in dy.host()], out_dt


@pytest.mark.parametrize("variant", [0, 8, 9])
@pytest.mark.parametrize("tx,tw", [(0, 0), (1, 0), (0, 1), (1, 1)])
@pytest.mark.parametrize("kk", [1, 8, 31, 33, 72, 95, 127, 168])
def test_bf16_any_reduction_length(kk, tx, tw, variant):
    """no whole stage, the remainder alone, fewer stages than the pipeline holds, and several rounds plus a remainder;
    one tile and a ragged second one of either tile size"""
    k, M, N = 2, 264, 136
    X, W = bf16(1, (M, k * kk)), bf16(2, (k * kk, N), 0.5)
    Xs, Ws = orc.scatter(X, orc.S1, k), orc.scatter(W, orc.S0, k)
    ref, _ = orc.matmul_sbp([values(x) for x in Xs], orc.S1, [values(w) for w in Ws], orc.S0)
    got, _ = run(Xs, orc.S1, Ws, orc.S0, M, k * kk, N, k, tx, tw, pitch(Xs, tx, 8), pitch(Ws, tw, 8), variant=variant)
    for i in range(k):
        assert_matmul_close(got[i], ref[i], 1e-5, f"kk={kk} trans=({tx},{tw}) v{variant} shard {i}")


@pytest.mark.parametrize("variant", [0, 40, 41, 42, 43, 44])
@pytest.mark.parametrize("aligned", [False, True])
@pytest.mark.parametrize("tx,tw", [(0, 0), (1, 0), (0, 1), (1, 1)])
@pytest.mark.parametrize("M,kk,N", [(1, 1, 1), (3, 5, 2), (31, 7, 9), (33, 65, 65), (64, 289, 64), (129, 544, 67), (140, 1000, 130)])
def test_bf16_any_shape_and_pitch(M, kk, N, tx, tw, aligned, variant):
    """no whole stage, one, fewer than waves, several per wave; rows shorter than a 16-byte chunk; odd pitches (register
    path) and 16-byte aligned ones (direct path)"""
    k = 2
    if variant == 40 and tx:
        pytest.skip("the 32-row tile takes a reduction-contiguous left operand")
    if variant == 42 and not aligned:
        pytest.skip("the 128 x 64 tile takes aligned rows")
    X, W = bf16(3, (M, k * kk)), bf16(4, (k * kk, N), 0.5)
    Xs, Ws = orc.scatter(X, orc.S1, k), orc.scatter(W, orc.S0, k)
    ref, _ = orc.matmul_sbp([values(x) for x in Xs], orc.S1, [values(w) for w in Ws], orc.S0)
    to, extra = (8, 0) if aligned else (2, 1)
    got, _ = run(Xs, orc.S1, Ws, orc.S0, M, k * kk, N, k, tx, tw, pitch(Xs, tx, to, extra), pitch(Ws, tw, to, extra), pitch(ref, 0, 2, 1), variant=variant)
    for i in range(k):
        assert_matmul_close(got[i], ref[i], 1e-5, f"{M}x{kk}x{N} trans=({tx},{tw}) v{variant} shard {i}")


@pytest.mark.parametrize("out", ["f32", "bf16", "gelu"])
@pytest.mark.parametrize("tx,tw", [(0, 0), (1, 0), (0, 1), (1, 1)])
@pytest.mark.parametrize("M,kk,N", [(1, 8, 1), (128, 64, 128), (130, 63, 129), (200, 128, 300), (129, 200, 136), (260, 1000, 140), (64, 449, 200)])
def test_bf16_two_wave_groups_over_the_reduction(M, kk, N, tx, tw, out):
    """variant 48: no whole 64-deep stage, one, two, fewer and more than the pipeline holds, with and without a remainder;
    one tile and ragged further ones"""
    k = 2
    if out == "f32":
        X, W, sx, sw, K, C = bf16(3, (M, k * kk)), bf16(4, (k * kk, N), 0.5), orc.S1, orc.S0, k * kk, N
    else:
        X, W, sx, sw, K, C = bf16(3, (M, kk)), bf16(4, (kk, k * N), 0.1), orc.B, orc.S1, kk, k * N
    Xs, Ws = orc.scatter(X, sx, k), orc.scatter(W, sw, k)
    ref, _ = orc.matmul_sbp([values(x) for x in Xs], sx, [values(w) for w in Ws], sw)
    epi = sbp.EPI_GELU if out == "gelu" else sbp.EPI_NONE
    got, _ = run(Xs, sx, Ws, sw, M, K, C, k, tx, tw, pitch(Xs, tx, 8), pitch(Ws, tw, 8), pitch(ref, 0, 2, 1), variant=48, epilogue=epi)
    for i in range(k):
        assert_matmul_close(got[i], orc.gelu(ref[i]) if out == "gelu" else ref[i], 1e-5 if out == "f32" else 2.0 ** -7, f"{M}x{kk}x{N} trans=({tx},{tw}) {out} shard {i}")


@pytest.mark.parametrize("tx,tw", [(0, 0), (1, 0), (0, 1), (1, 1)])
@pytest.mark.parametrize("M,kk,N,extra,start", [(130, 64, 129, 8, 0), (128, 72, 200, 24, 56), (140, 200, 136, 0, 8), (260, 256, 130, 40, 24), (129, 330, 257, 8, 120),
                                                (300, 3300, 140, 16, 64), (256, 2113, 384, 56, 40), (140, 3136, 256, 0, 0)])
def test_bf16_rows_anywhere_in_a_cache_line(M, kk, N, extra, start, tx, tw):
    """variant 48, buffers that start and rows that lie 16-byte aligned anywhere in a 128-byte line, or all on lines: one stage to more
    than the pipeline holds, with and without a remainder; NaN before, between and behind the rows"""
    import torch
    k = 2
    X, W = bf16(3, (M, k * kk)), bf16(4, (k * kk, N), 0.5)
    Xs, Ws = orc.scatter(X, orc.S1, k), orc.scatter(W, orc.S0, k)
    ref, _ = orc.matmul_sbp([values(x) for x in Xs], orc.S1, [values(w) for w in Ws], orc.S0)
    keep = []

    def place(shards, trans):
        ld = pitch(shards, trans, 8, extra)
        ptrs = []
        for a in (s.T if trans else s for s in shards):
            buf = torch.full((start + a.shape[0] * ld,), 0x7FC1, dtype=torch.int16, device="cuda")
            buf[start:].view(a.shape[0], ld)[:, :a.shape[1]] = torch.from_numpy(np.ascontiguousarray(a).view(np.int16)).cuda()
            keep.append(buf)
            ptrs.append(buf.data_ptr() + 2 * start)
        return ptrs, ld

    (px, ldx), (pw, ldw) = place(Xs, tx), place(Ws, tw)
    dy = DevTensor.empty(M, N, np.float32, orc.P_SUM, k)
    sbp.sbp_set_knob(sbp.KNOB_GEMM_VARIANT, 48)
    try:
        sbp.sbp_matmul(sbp.SbpTensor(px, M, k * kk, sbp.BF16, tx, ldx), sbp.S(1), sbp.SbpTensor(pw, k * kk, N, sbp.BF16, tw, ldw), sbp.S(0), dy.desc, sbp.AUTO, k)
        sync()
    finally:
        sbp.sbp_set_knob(sbp.KNOB_GEMM_VARIANT, 0)
    for i, y in enumerate(dy.host()):
        assert_matmul_close(y, ref[i], 1e-5, f"{M}x{kk}x{N} trans=({tx},{tw}) shard {i}")


def on_device(seed, shapes, trans, extra=0, start=0, scale=1.0):
    """buffers of random bf16 on the device, rows of a pitch that is a multiple of 8, `start` elements into an allocation; NaN around
    them.  The matrices, what keeps them, and pointers and pitch for a descriptor"""
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)
    ld = -(-max(r if trans else c for r, c in shapes) // 8) * 8 + extra
    mats, keep = [], []
    for r, c in shapes:
        stored = (c, r) if trans else (r, c)
        buf = torch.full((start + stored[0] * ld,), float("nan"), dtype=torch.bfloat16, device="cuda")
        view = buf[start:].view(stored[0], ld)[:, :stored[1]]
        view.normal_(0.0, scale, generator=g)
        keep.append(buf)
        mats.append(view.T if trans else view)
    return mats, keep, [b.data_ptr() + 2 * start for b in keep], ld


def close_on_device(y, x, w, gelu, bar):
    import torch
    ref = x.float() @ w.float()
    if gelu:
        ref = torch.nn.functional.gelu(ref)
    y = y.float()
    return bool((torch.abs(y - ref) <= bar * torch.maximum(ref.abs(), ref.square().mean().sqrt())).all())


@pytest.mark.parametrize("tx,tw", [(0, 0), (1, 0), (0, 1), (1, 1)])
@pytest.mark.parametrize("k,M,N,kk,extra,start", [(8, 1024, 512, 11008, 0, 0), (8, 1000, 499, 11200, 24, 40), (8, 1020, 450, 11463, 8, 64), (4, 1001, 1023, 16640, 0, 0)])
def test_bf16_lines_touched_ahead(k, M, N, kk, extra, start, tx, tw):
    """variant 48 on operands of more than 256 MiB whose shards each lie on one XCD (8 x 4 tiles: shares of 512 / 4 + 512 / 8 lines) or
    half of one (bands of 4 x 8 tiles): every workgroup touches its share ahead; whole and cut tiles, rows on lines and anywhere"""
    import torch
    xs, keepx, px, ldx = on_device(SEED + 61, [(M, kk)] * k, tx, extra, start)
    ws, keepw, pw, ldw = on_device(SEED + 62, [(kk, N)] * k, tw, extra, start, 0.5)
    assert 2 * k * kk * (M + N) > 256 << 20
    ys = [torch.full((M, N), float("nan"), device="cuda") for _ in range(k)]
    sbp.sbp_set_knob(sbp.KNOB_GEMM_VARIANT, 48)
    try:
        sbp.sbp_matmul(sbp.SbpTensor(px, M, k * kk, sbp.BF16, tx, ldx), sbp.S(1), sbp.SbpTensor(pw, k * kk, N, sbp.BF16, tw, ldw), sbp.S(0), sbp.SbpTensor(ys, M, N, sbp.F32), sbp.AUTO, k)
        sync()
    finally:
        sbp.sbp_set_knob(sbp.KNOB_GEMM_VARIANT, 0)
    # both sums run in fp32, in different orders: sqrt(kk) 2^-24 of the scale each, below 1e-5
    for i in range(k):
        assert close_on_device(ys[i], xs[i], ws[i], False, 2e-5), f"shard {i}"


@pytest.mark.parametrize("M", [32641, 32900])
def test_bf16_more_tile_rows_than_a_band_counts(M):
    """variant 48, eight devices of 256 and 258 tile-rows"""
    k, kk, N = 8, 72, 40
    X, W = bf16(3, (M, k * kk)), bf16(4, (k * kk, N), 0.5)
    Xs, Ws = orc.scatter(X, orc.S1, k), orc.scatter(W, orc.S0, k)
    got, _ = run(Xs, orc.S1, Ws, orc.S0, M, k * kk, N, k, 0, 0, pitch(Xs, 0, 8), pitch(Ws, 0, 8), variant=48)
    for i in range(k):
        assert_matmul_close(got[i], values(Xs[i]) @ values(Ws[i]), 1e-5, f"shard {i}")


@pytest.mark.parametrize("out", ["f32", "bf16", "gelu", "rowmax"])
@pytest.mark.parametrize("tx,tw", [(0, 0), (1, 0), (0, 1), (1, 1)])
@pytest.mark.parametrize("kk,ldy", [(128, 0), (256, 4352 + 8), (640, 4352 + 1)])
def test_bf16_persistent_tiles(kk, ldy, tx, tw, out):
    """variant 16, more 256 x 256 tiles than workgroups: tile after tile through one pipeline, with one round of stages, two and
    more, whole and cut tiles, rows of the result on cache lines, 16-byte aligned and odd; against torch in fp32"""
    import torch
    k, M, N = 2, 2200, 4352
    X, W = bf16(21, (M, kk)), bf16(22, (kk, k * N), 0.1)
    Xs, Ws = orc.scatter(X, orc.B, k), orc.scatter(W, orc.S1, k)
    if out == "f32":
        X = bf16(21, (M, k * kk))
        W = bf16(22, (k * kk, N), 0.1)
        Xs, Ws = orc.scatter(X, orc.S1, k), orc.scatter(W, orc.S0, k)
    sx, sw, K, C = (orc.S1, orc.S0, k * kk, N) if out == "f32" else (orc.B, orc.S1, kk, k * N)
    dx = DevTensor.from_host(Xs, M, K, sx, trans=tx, ld=pitch(Xs, tx, 8))
    dw = DevTensor.from_host(Ws, K, C, sw, trans=tw, ld=pitch(Ws, tw, 8))
    dy = DevTensor.empty(M, C, np.float32 if out == "f32" else np.uint16, orc.P_SUM if out == "f32" else orc.S1, k, ld=ldy)
    dm = DevTensor.empty(M, 1, np.float32, orc.P_MAX, k)
    sbp.sbp_set_knob(sbp.KNOB_GEMM_VARIANT, 16)
    try:
        if out == "rowmax":
            sbp.sbp_matmul_rowmax(dx.desc, TO_ABI[sx], dw.desc, TO_ABI[sw], dy.desc, sbp.AUTO, dm.desc, k)
        else:
            sbp.sbp_matmul_ex(dx.desc, TO_ABI[sx], dw.desc, TO_ABI[sw], dy.desc, sbp.AUTO, k, None, sbp.EPI_GELU if out == "gelu" else sbp.EPI_NONE)
        sync()
    finally:
        sbp.sbp_set_knob(sbp.KNOB_GEMM_VARIANT, 0)
    got, top = dy.host(), dm.host()
    for i in range(k):
        ref = (torch.from_numpy(values(Xs[i]).astype(np.float32)).cuda() @ torch.from_numpy(values(Ws[i]).astype(np.float32)).cuda()).cpu().numpy()
        if out == "gelu":
            ref = orc.gelu(ref)
        y = got[i] if out == "f32" else values(got[i])
        assert_matmul_close(y, ref, 1e-5 if out == "f32" else 2.0 ** -7, f"kk={kk} ldy={ldy} trans=({tx},{tw}) {out} shard {i}")
        if out == "rowmax":
            assert np.array_equal(top[i][:, 0], y.max(axis=1))


@pytest.mark.parametrize("variant", [16, 21])
@pytest.mark.parametrize("out", ["f32", "bf16", "gelu", "rowmax"])
@pytest.mark.parametrize("kk,tx,tw", [(128, 0, 0), (128, 1, 1), (384, 0, 1), (384, 1, 0)])
@pytest.mark.parametrize("N", [301, 392, 515])
def test_bf16_tiles_after_cut_ones(N, kk, tx, tw, out, variant):
    """two devices of 130 tile-rows, every second or third tile cut by the last column (inside 16 bytes or not), more than two tiles a
    workgroup: what is counted of a cut tile's stores when the next tile's stages are waited for"""
    import torch
    k, M = 2, 33100
    sx, sw, K, C = (sbp.S(1), sbp.S(0), k * kk, N) if out == "f32" else (sbp.B, sbp.S(1), kk, k * N)
    xs, keepx, px, ldx = on_device(SEED + 63, [(M, kk)] * k, tx)
    if out != "f32":
        xs, px = [xs[0]] * k, [px[0]] * k
    ws, keepw, pw, ldw = on_device(SEED + 64, [(kk, N)] * k, tw, scale=0.1)
    ldy = N + 3
    bufs = [torch.full((M, ldy), 777.0, dtype=torch.float32 if out == "f32" else torch.bfloat16, device="cuda") for _ in range(k)]
    tops = [torch.full((M,), float("nan"), device="cuda") for _ in range(k)]
    X, W = sbp.SbpTensor(px, M, K, sbp.BF16, tx, ldx), sbp.SbpTensor(pw, K, C, sbp.BF16, tw, ldw)
    Y = sbp.SbpTensor(bufs, M, C, sbp.F32 if out == "f32" else sbp.BF16, 0, ldy)
    sbp.sbp_set_knob(sbp.KNOB_GEMM_VARIANT, variant)
    try:
        if out == "rowmax":
            sbp.sbp_matmul_rowmax(X, sx, W, sw, Y, sbp.AUTO, sbp.SbpTensor(tops, M, 1, sbp.F32), k)
        else:
            sbp.sbp_matmul_ex(X, sx, W, sw, Y, sbp.AUTO, k, None, sbp.EPI_GELU if out == "gelu" else sbp.EPI_NONE)
        sync()
    finally:
        sbp.sbp_set_knob(sbp.KNOB_GEMM_VARIANT, 0)
    for i in range(k):
        assert close_on_device(bufs[i][:, :N], xs[i], ws[i], out == "gelu", 1e-5 if out == "f32" else 2.0 ** -7), f"shard {i}"
        assert bool((bufs[i][:, N:] == 777.0).all()), f"shard {i}: padding written"
        if out == "rowmax":
            assert bool((tops[i] == bufs[i][:, :N].float().amax(1)).all())


@pytest.mark.parametrize("variant", [8, 9, 16, 21])
@pytest.mark.parametrize("out", ["f32", "bf16", "gelu", "rowmax"])
@pytest.mark.parametrize("M,N,odd", [(255, 264, 0), (300, 388, 1), (257, 392, 0), (130, 391, 0), (140, 389, 1), (512, 520, 3),
                                     (129, 385, 0), (161, 394, 1), (225, 163, 0), (130, 190, 1), (289, 141, 3), (300, 13, 0), (81, 9, 1)])
def test_bf16_tiles_cut_by_the_edge(M, N, odd, out, variant):
    """results stored 16 bytes at a time up to the edge: rows cut anywhere, columns at a multiple of 16 bytes or inside one, rows at any
    pitch; the padding behind a row stays as it was (DevTensor)"""
    k, kk = 2, 256
    if out == "f32":
        X, W, sx, sw, K, C = bf16(3, (M, k * kk)), bf16(4, (k * kk, N), 0.5), orc.S1, orc.S0, k * kk, N
    else:
        X, W, sx, sw, K, C = bf16(3, (M, kk)), bf16(4, (kk, k * N), 0.1), orc.B, orc.S1, kk, k * N
    Xs, Ws = orc.scatter(X, sx, k), orc.scatter(W, sw, k)
    ref, _ = orc.matmul_sbp([values(x) for x in Xs], sx, [values(w) for w in Ws], sw)
    dx, dw = DevTensor.from_host(Xs, M, K, sx, ld=kk), DevTensor.from_host(Ws, K, C, sw, ld=-(-N // 8) * 8)
    dy = DevTensor.empty(M, C, np.float32 if out == "f32" else np.uint16, orc.P_SUM if out == "f32" else orc.S1, k, ld=-(-N // 8) * 8 + 8 + odd)
    dm = DevTensor.empty(M, 1, np.float32, orc.P_MAX, k)
    sbp.sbp_set_knob(sbp.KNOB_GEMM_VARIANT, variant)
    try:
        if out == "rowmax":
            sbp.sbp_matmul_rowmax(dx.desc, TO_ABI[sx], dw.desc, TO_ABI[sw], dy.desc, sbp.AUTO, dm.desc, k)
        else:
            sbp.sbp_matmul_ex(dx.desc, TO_ABI[sx], dw.desc, TO_ABI[sw], dy.desc, sbp.AUTO, k, None, sbp.EPI_GELU if out == "gelu" else sbp.EPI_NONE)
        sync()
    finally:
        sbp.sbp_set_knob(sbp.KNOB_GEMM_VARIANT, 0)
    got, top = dy.host(), dm.host()
    for i in range(k):
        y = got[i] if out == "f32" else values(got[i])
        assert_matmul_close(y, orc.gelu(ref[i]) if out == "gelu" else ref[i], 1e-5 if out == "f32" else 2.0 ** -7, f"{M}x{N} {out} v{variant} shard {i}")
        if out == "rowmax":
            assert np.array_equal(top[i][:, 0], y.max(axis=1))


@pytest.mark.parametrize("variant", [0, 51, 52])
@pytest.mark.parametrize("odd", [0, 1])
@pytest.mark.parametrize("M,kk,N", [(1, 1, 1), (3, 255, 2), (32, 256, 32), (33, 263, 31), (64, 511, 65), (70, 512, 40), (31, 777, 130), (130, 1025, 64), (65, 9000, 70),
                                    (9, 258, 33), (40, 259, 9), (5, 260, 34), (33, 261, 5), (17, 518, 40)])
def test_bf16_long_pieces_of_rows(M, kk, N, odd, variant):
    """both operands reduction-contiguous, fp32 results: no whole 256-deep stage, one, two, three and more, with and without a remainder;
    rows of any pitch; one tile and ragged further ones"""
    k = 2
    X, W = bf16(3, (M, k * kk)), bf16(4, (k * kk, N), 0.5)
    Xs, Ws = orc.scatter(X, orc.S1, k), orc.scatter(W, orc.S0, k)
    ref, _ = orc.matmul_sbp([values(x) for x in Xs], orc.S1, [values(w) for w in Ws], orc.S0)
    got, _ = run(Xs, orc.S1, Ws, orc.S0, M, k * kk, N, k, 0, 1, pitch(Xs, 0, 8, odd), pitch(Ws, 1, 8, 8 + odd), pitch(ref, 0, 2, 1), variant=variant)
    for i in range(k):
        assert_matmul_close(got[i], ref[i], 1e-5, f"{M}x{kk}x{N} odd={odd} v{variant} shard {i}")


@pytest.mark.parametrize("epilogue", [sbp.EPI_NONE, sbp.EPI_GELU])
@pytest.mark.parametrize("M,K,N", [(5, 33, 7), (70, 100, 203)])
def test_bf16_odd_rows_rounded_results(M, K, N, epilogue):
    k = 3
    X, W = bf16(5, (M, K)), bf16(6, (K, N), 0.2)
    Xs, Ws = orc.scatter(X, orc.B, k), orc.scatter(W, orc.S1, k)
    ref, _ = orc.matmul_sbp([values(x) for x in Xs], orc.B, [values(w) for w in Ws], orc.S1)
    got, _ = run(Xs, orc.B, Ws, orc.S1, M, K, N, k, 0, 0, 0, 0, epilogue=epilogue)
    for i in range(k):
        r = orc.gelu(ref[i]) if epilogue == sbp.EPI_GELU else ref[i]
        assert_matmul_close(got[i], r, 2.0 ** -7, f"epilogue {epilogue} shard {i}")


def f32(tid, shape):
    return wl.uniform(SEED, tid, shape).astype(np.float32)


@pytest.mark.parametrize("variant", [0, 45, 46, 47])
@pytest.mark.parametrize("tx,tw", [(0, 0), (1, 0), (0, 1), (1, 1)])
@pytest.mark.parametrize("types", ["f32,f32", "f32,bf16", "bf16,f32"])
@pytest.mark.parametrize("M,kk,N", [(1, 1, 1), (3, 5, 2), (31, 15, 9), (33, 65, 66), (64, 128, 64), (129, 131, 67), (140, 321, 257)])
def test_f32_operands_any_shape_and_pitch(M, kk, N, types, tx, tw, variant):
    """the fp32 matrix instruction: no whole stage, one, several and a remainder, rows shorter than a chunk, one tile and
    a ragged second one of every tile size, fp32 x fp32 and either operand bf16.  Bar: summation order (see above)."""
    k = 2
    if types == "f32,f32":
        X, W, sx, sw = f32(7, (M, k * kk)), f32(8, (k * kk, N)), orc.S1, orc.S0
        Xs, Ws = orc.scatter(X, sx, k), orc.scatter(W, sw, k)
    elif types == "f32,bf16":
        X, W, sx, sw, kk = None, bf16(8, (kk, N), 0.5), orc.P_SUM, orc.B, kk
        Xs, Ws = [f32(10 + i, (M, kk)) for i in range(k)], orc.scatter(W, sw, k)
    else:
        X, W, sx, sw = bf16(7, (M, kk)), None, orc.B, orc.P_SUM
        Xs, Ws = orc.scatter(X, sx, k), [f32(10 + i, (kk, N)) for i in range(k)]
    wide = lambda v: values(v) if v.dtype == np.uint16 else v
    ref, _ = orc.matmul_sbp([wide(x) for x in Xs], sx, [wide(w) for w in Ws], sw)
    got, _ = run(Xs, sx, Ws, sw, M, k * kk if sx == orc.S1 else kk, N, k, tx, tw, pitch(Xs, tx, 2, 1), pitch(Ws, tw, 2, 1), pitch(ref, 0, 2, 1), variant=variant)
    for i in range(k):
        assert_matmul_close(got[i], ref[i], 1e-5, f"{M}x{kk}x{N} {types} trans=({tx},{tw}) v{variant} shard {i}")


@pytest.mark.parametrize("variant", [49, 50])
@pytest.mark.parametrize("tx,tw", [(0, 0), (1, 0), (0, 1), (1, 1)])
@pytest.mark.parametrize("types", ["f32,f32", "f32,bf16", "bf16,f32"])
@pytest.mark.parametrize("M,kk,N", [(1, 1, 1), (3, 31, 2), (33, 65, 66), (64, 32, 64), (129, 131, 67), (140, 321, 257), (128, 96, 136)])
def test_f32_operands_as_bf16_terms(M, kk, N, types, tx, tw, variant):
    """no whole 32-deep stage, one, several and a remainder, rows shorter than a chunk, one tile and ragged further ones.  Bar: the
    dropped products of terms are below 2^-25 of each product, the rest is summation order"""
    k = 2
    if types == "f32,f32":
        X, W, sx, sw = f32(7, (M, k * kk)), f32(8, (k * kk, N)), orc.S1, orc.S0
        Xs, Ws = orc.scatter(X, sx, k), orc.scatter(W, sw, k)
    elif types == "f32,bf16":
        W, sx, sw = bf16(8, (kk, N), 0.5), orc.P_SUM, orc.B
        Xs, Ws = [f32(10 + i, (M, kk)) for i in range(k)], orc.scatter(W, sw, k)
    else:
        X, sx, sw = bf16(7, (M, kk)), orc.B, orc.P_SUM
        Xs, Ws = orc.scatter(X, sx, k), [f32(10 + i, (kk, N)) for i in range(k)]
    wide = lambda v: values(v) if v.dtype == np.uint16 else v
    ref, _ = orc.matmul_sbp([wide(x) for x in Xs], sx, [wide(w) for w in Ws], sw)
    got, _ = run(Xs, sx, Ws, sw, M, k * kk if sx == orc.S1 else kk, N, k, tx, tw, pitch(Xs, tx, 2, 1), pitch(Ws, tw, 2, 1), pitch(ref, 0, 2, 1), variant=variant)
    for i in range(k):
        assert_matmul_close(got[i], ref[i], 1e-5, f"{M}x{kk}x{N} {types} trans=({tx},{tw}) v{variant} shard {i}")


@pytest.mark.parametrize("variant", [49, 50])
@pytest.mark.parametrize("types", ["f32,f32", "f32,bf16"])
@pytest.mark.parametrize("case", ["inf", "nan", "inf times zero", "lowest", "past the largest bf16", "overflow", "small", "denormal", "zero"])
def test_f32_values_that_terms_do_not_hold(case, types, variant):
    """values whose bf16 terms are not finite or lose bits: infinities, NaN and overflow where the fp32 instruction gives them (one tile
    of several), and the same accuracy; results in the range of fp32 denormals to one of their steps per product"""
    k, M, kk, N = 1, 140, 70, 150
    X, W = f32(31, (M, kk)), f32(32, (kk, N))
    if types == "f32,bf16":
        W = wl.to_bf16_bits(W)
    tiny = np.float32(2.0) ** -140
    if case == "inf":
        X[3, 5], X[135, 0] = np.inf, -np.inf
    elif case == "nan":
        X[77, 69] = np.nan
    elif case == "inf times zero":
        X[3, 5] = np.inf
        W[5, 7] = 0
    elif case == "lowest":
        X[9, :] = np.finfo(np.float32).min
    elif case == "past the largest bf16":
        X[130, 11], X[130, 12] = 3.4e38, -3.4e38
        W[11:13, :] = wl.to_bf16_bits(np.full((2, N), 0.25)) if types == "f32,bf16" else 0.25
    elif case == "overflow":   # in whatever order the sum is taken
        X[0, :4] = 3e38
        W[:4, :] = wl.to_bf16_bits(np.ones((4, N))) if types == "f32,bf16" else 1.0
    elif case == "small":
        X *= np.float32(1e-35)
        if types == "f32,f32":
            W *= np.float32(1e10)
    elif case == "denormal":
        X *= tiny
    elif case == "zero":
        X[:] = 0
    sx, sw = (orc.S1, orc.S0) if types == "f32,f32" else (orc.P_SUM, orc.B)
    got, _ = run([X], sx, [W], sw, M, kk, N, k, 0, 0, 0, 0, variant=variant)
    want, _ = run([X], sx, [W], sw, M, kk, N, k, 0, 0, 0, 0, variant=45)
    wide = (values(W) if W.dtype == np.uint16 else W).astype(np.float64)
    got, want = got[0], want[0]
    assert np.array_equal(np.isnan(got), np.isnan(want)) and np.array_equal(np.isposinf(got), np.isposinf(want)) and np.array_equal(np.isneginf(got), np.isneginf(want))
    with np.errstate(all="ignore"):
        ref = X.astype(np.float64) @ wide
        scale = np.abs(X.astype(np.float64)) @ np.abs(wide)
    ok = np.isfinite(want)
    assert np.all(np.abs(got[ok] - ref[ok]) <= 1e-5 * scale[ok] + kk * 2.0 ** -149)


@pytest.mark.parametrize("variant,M,kk,N", [(49, 140, 70, 150), (50, 140, 70, 150), (0, 2046, 300, 2050)])
@pytest.mark.parametrize("tx,tw", [(0, 0), (1, 0), (0, 1), (1, 1)])
@pytest.mark.parametrize("types", ["f32,f32", "f32,bf16", "bf16,f32"])
@pytest.mark.parametrize("e", [-110, -111, -118, -126, -140])
def test_f32_small_values_beside_ordinary_ones(e, types, tx, tw, variant, M, kk, N):
    """one row of X, one column of W and one value of each that are 2^e in size among ordinary ones of 2^50, so that their results are
    ordinary numbers: every result to the accuracy that fp32 operands give it.  From 2^-110 on down the bf16 terms cannot hold
    fp32's bits"""
    k = 1
    X, W = (wl.uniform(SEED, t, shape, 1.0, 2.0).astype(np.float32) for t, shape in ((41, (M, kk)), (42, (kk, N))))
    S, tiny = np.float32(2.0) ** 50, np.float32(2.0) ** e
    X *= S
    W *= S
    if types != "bf16,f32":
        X[5], X[99] = X[5] / S * tiny, 0
        X[99, 33] = 1.1 * tiny
    if types != "f32,bf16":
        W[:, 7], W[:, 91] = W[:, 7] / S * tiny, 0
        W[41, 91] = 1.1 * tiny
    if types == "f32,f32":
        sx, sw = orc.S1, orc.S0
    else:
        sx, sw = (orc.P_SUM, orc.B) if types == "f32,bf16" else (orc.B, orc.P_SUM)
        X, W = (X, wl.to_bf16_bits(W)) if types == "f32,bf16" else (wl.to_bf16_bits(X), W)
    got, _ = run([X], sx, [W], sw, M, kk, N, k, tx, tw, pitch([X], tx, 2, 1), pitch([W], tw, 2, 1), variant=variant)
    x, w = values(X), values(W)
    ref, scale = x @ w, np.abs(x) @ np.abs(w)
    bad = np.abs(got[0] - ref) > 1e-5 * scale + kk * 2.0 ** -149
    assert not bad.any(), f"{bad.sum()} results off, rows {np.unique(np.nonzero(bad)[0])[:8]}, columns {np.unique(np.nonzero(bad)[1])[:8]}"


@pytest.mark.parametrize("variant", [0, 49, 50])
@pytest.mark.parametrize("types", ["f32,bf16", "bf16,f32"])
def test_f32_next_to_small_bf16_values(types, variant):
    """one row or column of bf16 denormals next to fp32 values of 2^60"""
    M, kk, N = 140, 70, 150
    X, W = (wl.uniform(SEED, t, shape, 1.0, 2.0).astype(np.float32) for t, shape in ((45, (M, kk)), (46, (kk, N))))
    if types == "f32,bf16":
        X *= np.float32(2.0) ** 60
        W[:, 7] *= np.float32(2.0) ** -130
        W, sx, sw = wl.to_bf16_bits(W), orc.P_SUM, orc.B
    else:
        W *= np.float32(2.0) ** 60
        X[5] *= np.float32(2.0) ** -130
        X, sx, sw = wl.to_bf16_bits(X), orc.B, orc.P_SUM
    got, _ = run([X], sx, [W], sw, M, kk, N, 1, 0, 0, pitch([X], 0, 2, 1), pitch([W], 0, 2, 1), variant=variant)
    ref = values(X) @ values(W)
    assert np.all(ref > 0) and np.all(np.abs(got[0] - ref) <= 1e-5 * ref)


@pytest.mark.parametrize("variant", [49, 50])
def test_f32_small_values_cost_no_second_multiplication(variant):
    """the tail of a softmax (one value in fifty between 2^-149 and 2^-111) is held by the terms: as fast as ordinary values.  Multiplying
    every tile again on the fp32 instruction takes 2.2 times as long; 1.4 leaves room for the clock"""
    import torch
    M = kk = N = 2048
    g = torch.Generator(device="cuda").manual_seed(SEED)
    x, w = (torch.empty((M, kk), device="cuda").normal_(generator=g) for _ in range(2))
    tail = x * torch.exp2(torch.randint(-149, -111, x.shape, device="cuda", generator=g).float())
    xs = torch.where(torch.rand(x.shape, device="cuda", generator=g) < 0.02, tail, x)
    y = torch.empty((M, N), device="cuda")
    ty, tw, tx = sbp.SbpTensor([y], M, N, sbp.F32), sbp.SbpTensor([w], kk, N, sbp.F32), [sbp.SbpTensor([t], M, kk, sbp.F32) for t in (x, xs)]
    best = [float("inf"), float("inf")]
    sbp.sbp_set_knob(sbp.KNOB_GEMM_VARIANT, variant)
    try:
        for _ in range(6):
            for i, t in enumerate(tx):
                a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                a.record()
                for _ in range(5):
                    sbp.sbp_matmul(t, sbp.S(1), tw, sbp.S(0), ty, sbp.AUTO, 1)
                b.record()
                sync()
                best[i] = min(best[i], a.elapsed_time(b))
    finally:
        sbp.sbp_set_knob(sbp.KNOB_GEMM_VARIANT, 0)
    assert best[1] <= 1.4 * best[0], best


@pytest.mark.parametrize("variant", [49, 50])
@pytest.mark.parametrize("small", [False, True])
@pytest.mark.parametrize("M,kk,N", [(130, 70, 203), (5, 40, 6), (129, 65, 64)])
def test_f32_terms_and_what_lies_behind_the_rows(M, kk, N, small, variant):
    """both operands reduction-major, widths that are no multiple of 8: NaN, tiny and large values in the padding between rows give the
    same bits, for ordinary and for small operands"""
    import torch
    X, W = f32(43, (M, kk)), f32(44, (kk, N))
    if small:
        X *= np.float32(2.0) ** -118
        W *= np.float32(2.0) ** 60
    out = []
    for behind in (np.nan, 1e-41, 1e30, 0.0):
        bufs = []
        for a in (np.ascontiguousarray(X.T), W):
            buf = torch.full((a.shape[0], a.shape[1] + 9), float(behind), device="cuda")
            buf[:, :a.shape[1]] = torch.from_numpy(a).cuda()
            bufs.append(buf)
        dy = DevTensor.empty(M, N, np.float32, orc.P_SUM, 1)
        sbp.sbp_set_knob(sbp.KNOB_GEMM_VARIANT, variant)
        try:
            sbp.sbp_matmul(sbp.SbpTensor([bufs[0]], M, kk, sbp.F32, 1, M + 9), sbp.S(1), sbp.SbpTensor([bufs[1]], kk, N, sbp.F32, 0, N + 9), sbp.S(0), dy.desc, sbp.AUTO, 1)
            sync()
        finally:
            sbp.sbp_set_knob(sbp.KNOB_GEMM_VARIANT, 0)
        out.append(dy.host()[0])
    x, w = X.astype(np.float64), W.astype(np.float64)
    assert np.all(np.abs(out[0] - x @ w) <= 1e-5 * (np.abs(x) @ np.abs(w)))
    assert all(np.array_equal(o, out[0]) for o in out[1:])


@pytest.mark.parametrize("M,K,N", [(5, 33, 7), (70, 300, 203)])
def test_f32_gelu(M, K, N):
    k = 3
    X, W = f32(5, (M, K)), f32(6, (K, N))
    Xs, Ws = orc.scatter(X, orc.B, k), orc.scatter(W, orc.S1, k)
    ref, _ = orc.matmul_sbp(Xs, orc.B, Ws, orc.S1)
    got, _ = run(Xs, orc.B, Ws, orc.S1, M, K, N, k, 0, 0, 0, 0, epilogue=sbp.EPI_GELU)
    for i in range(k):
        assert_matmul_close(got[i], orc.gelu(ref[i]), 1e-5, f"gelu shard {i}")


@pytest.mark.parametrize("tx", [0, 1])
@pytest.mark.parametrize("K", [256, 200])
def test_row_maxima_under_every_forced_kernel(K, tx):
    """sbp_matmul_rowmax under every knob value: a forced kernel that cannot write row maxima is followed by the row
    reduction, one that cannot take the shape refuses.  The maxima are those of the stored values, exactly."""
    k, M, N = 2, 264, 2 * 200
    X, W = bf16(20, (M, K)), bf16(21, (K, N), 0.2)
    Xs, Ws = orc.scatter(X, orc.B, k), orc.scatter(W, orc.S1, k)
    ref, _ = orc.matmul_sbp([values(x) for x in Xs], orc.B, [values(w) for w in Ws], orc.S1)
    dx, dw = DevTensor.from_host(Xs, M, K, orc.B, trans=tx), DevTensor.from_host(Ws, K, N, orc.S1)
    ran = set()
    for variant in range(64):
        dy, dm = DevTensor.empty(M, N, np.uint16, orc.S1, k), DevTensor.empty(M, 1, np.float32, orc.P_MAX, k)
        sbp.sbp_set_knob(sbp.KNOB_GEMM_VARIANT, variant)
        try:
            sbp.sbp_matmul_rowmax(dx.desc, sbp.B, dw.desc, sbp.S(1), dy.desc, sbp.AUTO, dm.desc, k)
        except sbp.SbpError as e:
            assert e.status == -9, f"variant {variant}: {e}"
            continue
        finally:
            sbp.sbp_set_knob(sbp.KNOB_GEMM_VARIANT, 0)
        sync()
        ran.add(variant)
        for i, (y, m) in enumerate(zip(dy.host(), dm.host())):
            assert_matmul_close(values(y), ref[i], 2.0 ** -7, f"K={K} v{variant} shard {i}")
            assert np.array_equal(m[:, 0].astype(np.float64), values(y).max(axis=1)), f"K={K} v{variant}: row maxima of shard {i}"
    assert {0, 1, 8, 9, 41, 42, 43, 44, 48} <= ran


@pytest.mark.parametrize("K,to,extra,variant", [(K, 8, 0, v) for K in (1, 40, 1000) for v in (0, 8, 9, 40, 41, 42, 43, 44, 48)]
                         + [(K, 2, 1, v) for K in (1, 1000, 4100) for v in (0, 40, 41, 43, 44)])   # 8, 9, 42, 48 take aligned rows
def test_gelu_keeps_fp32_accuracy_where_the_reduction_fits_no_step(K, to, extra, variant):
    """One product per element, exact in fp32, so that only GeLU and the rounding to bf16 are left.  Bound: half a step of
    the result plus 2^-18 of it.  For |x| <= 4 erfc's argument z = |x| / sqrt 2 is off by 2^-23 of itself at most (the
    constant, the product), which erfc magnifies 2 z^2 + 1 <= 17 times to 2.0e-6; erfcf's 4 ulp and two products add
    0.6e-6; 2^-18 is 3.8e-6.  (A fit good to 2.2e-5 leaves several elements of these outside.)  NaN stays NaN."""
    k, M, N = 2, 300, 2 * 160
    X, W = np.zeros((M, K), np.uint16), wl.to_bf16_bits(np.zeros((K, N)))
    X[:, 0] = wl.to_bf16_bits(wl.uniform(SEED, 22, (M, 1), -2.0, -0.25))[:, 0]
    W[0] = wl.to_bf16_bits(wl.uniform(SEED, 23, (1, N), 0.25, 2.0))[0]
    X[7, 0] = 0x7FC0
    Xs, Ws = orc.scatter(X, orc.B, k), orc.scatter(W, orc.S1, k)
    got, _ = run(Xs, orc.B, Ws, orc.S1, M, K, N, k, 0, 0, pitch(Xs, 0, to, extra), pitch(Ws, 0, to, extra), variant=variant, epilogue=sbp.EPI_GELU)
    for i in range(k):
        x = values(X[:, :1]) * values(Ws[i][:1])
        ok = np.arange(M) != 7
        assert np.isnan(got[i][7]).all(), "NaN"
        ref = orc.gelu(x[ok])
        step = 2.0 ** (np.floor(np.log2(np.abs(ref))) - 7)
        bad = np.abs(got[i][ok] - ref) > 0.5 * step + 2.0 ** -18 * np.abs(ref)
        assert not bad.any(), f"K={K} v{variant} shard {i}: {bad.sum()} of {bad.size} further off than rounding explains"


@pytest.mark.parametrize("variant", [0, 31, 32])
@pytest.mark.parametrize("extra", [0, 4])
@pytest.mark.parametrize("f32_side", ["x", "w"])
@pytest.mark.parametrize("n,kk", [(12, 32), (268, 96), (300, 256)])
def test_split_kernel_on_rows_that_end_inside_a_chunk(n, kk, f32_side, extra, variant):
    """an fp32 P(sum) operand stored along the reduction, its rows 8 i + 4 floats long, dense and with 4 floats of padding
    (NaN); the last chunk of a row is half of it.  Bar: summation order."""
    k, other = 2, 264
    if f32_side == "w":
        X, sx, sw, M, N, tx, tw = bf16(30, (other, kk)), orc.B, orc.P_SUM, other, n, 0, 0
        Xs, Ws = orc.scatter(X, sx, k), [f32(31 + i, (kk, n)) for i in range(k)]
    else:
        W, sx, sw, M, N, tx, tw = bf16(30, (kk, other), 0.5), orc.P_SUM, orc.B, n, other, 1, 0
        Xs, Ws = [f32(31 + i, (n, kk)) for i in range(k)], orc.scatter(W, sw, k)
    wide = lambda v: values(v) if v.dtype == np.uint16 else v
    ref, _ = orc.matmul_sbp([wide(x) for x in Xs], sx, [wide(w) for w in Ws], sw)
    ld = n + extra
    got, _ = run(Xs, sx, Ws, sw, M, kk, N, k, tx, tw, ld if f32_side == "x" else 0, ld if f32_side == "w" else 0, variant=variant)
    for i in range(k):
        assert_matmul_close(got[i], ref[i], 1e-5, f"{f32_side} {n}x{kk}+{extra} v{variant} shard {i}")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_more_tiles_than_a_launch_holds(dtype):
    """one row per device, 2^24 columns, 64 devices: 2^24 tiles of 64 x 64, 2^32 work items.  Single products: exact in fp32
    for bf16 operands, correctly rounded otherwise."""
    torch = __import__("torch")
    k, n, td = 64, 1 << 24, torch.float32 if dtype == "f32" else torch.bfloat16
    code = sbp.F32 if dtype == "f32" else sbp.BF16
    x = [torch.full((1, 1), 0.5 + i, dtype=td, device="cuda") for i in range(k)]
    w = torch.randn(1, n, device="cuda", dtype=td)
    y = [torch.full((1, n), float("nan"), dtype=td, device="cuda") for _ in range(k)]
    sbp.sbp_matmul(sbp.SbpTensor(x, k, 1, code), sbp.S(0), sbp.SbpTensor([w] * k, 1, n, code), sbp.B, sbp.SbpTensor(y, k, n, code), sbp.S(0), k)
    sync()
    for i in range(k):
        assert torch.equal(y[i], (x[i].float() * w.float()).to(td)), f"shard {i}"


@pytest.mark.parametrize("rows", [2 ** 31 - 1, 2 ** 31 - 64])
def test_extents_near_the_largest_are_refused(rows):
    """rounding such an extent up to tiles leaves 32 bits; the product is one that no kernel here takes"""
    torch = __import__("torch")
    x, y = (torch.empty(rows, 1, device="cuda") for _ in range(2))
    w = torch.ones(1, 1, device="cuda")
    with pytest.raises(sbp.SbpError) as e:
        sbp.sbp_matmul(sbp.SbpTensor([x], rows, 1, sbp.F32), sbp.B, sbp.SbpTensor([w], 1, 1, sbp.F32), sbp.B, sbp.SbpTensor([y], rows, 1, sbp.F32), sbp.B, 1)
    assert e.value.status == -9
    sync()


ROUNDED = [(v, a, tx, tw) for v in (0, 40, 41, 42, 43, 44) for a in (True, False) for tx in (0, 1) for tw in (0, 1)
           if not (v == 40 and tx) and not (v == 42 and not a)]   # 40: reduction-contiguous left operand; 42: aligned rows


@pytest.mark.parametrize("epilogue", [sbp.EPI_NONE, sbp.EPI_GELU])
@pytest.mark.parametrize("variant,aligned,tx,tw", ROUNDED)
@pytest.mark.parametrize("M,kk,N", [(1, 9, 3), (33, 65, 65), (64, 544, 72), (130, 1024, 131)])
def test_bf16_rounded_results_any_shape_and_pitch(M, kk, N, variant, aligned, tx, tw, epilogue):
    """results rounded to bf16, plain and under GeLU, at an odd row pitch: the additions of the waves' partial tiles, the
    store of eight columns a lane and its ragged ends.  Bar: one rounding, half a step
    of 8 significant bits, at most 2^-8 of the value, and the fp32 sums before it."""
    k = 2
    X, W = bf16(40, (M, kk)), bf16(41, (kk, k * N), 0.2)
    Xs, Ws = orc.scatter(X, orc.B, k), orc.scatter(W, orc.S1, k)
    ref, _ = orc.matmul_sbp([values(x) for x in Xs], orc.B, [values(w) for w in Ws], orc.S1)
    to, extra = (8, 0) if aligned else (2, 1)
    got, _ = run(Xs, orc.B, Ws, orc.S1, M, kk, k * N, k, tx, tw, pitch(Xs, tx, to, extra), pitch(Ws, tw, to, extra), pitch(ref, 0, 2, 1), variant=variant, epilogue=epilogue)
    for i in range(k):
        r = orc.gelu(ref[i]) if epilogue == sbp.EPI_GELU else ref[i]
        assert_matmul_close(got[i], r, 2.0 ** -8 + 1e-4, f"{M}x{kk}x{N} trans=({tx},{tw}) v{variant} epilogue {epilogue} shard {i}")


@pytest.mark.parametrize("epilogue", [sbp.EPI_NONE, sbp.EPI_GELU])
@pytest.mark.parametrize("k,M,kk,N,extra", [(8, 500, 37, 500, 1), (3, 1000, 640, 904, 0), (2, 40, 640, 1000, 0), (8, 72, 704, 4400, 0), (4, 100, 384, 3000, 0), (2, 1304, 200, 2000, 0)])
def test_bf16_rounded_results_default_choice(k, M, kk, N, extra, epilogue):
    """one shape for each kernel that the default choice takes for rounded results of these sizes: 128 x 128 tiles through
    registers, two wave groups over the reduction, the waves splitting it, two 64-deep stages (two shapes), four 32-deep ones"""
    X, W = bf16(42, (M, kk)), bf16(43, (kk, k * N), 0.2)
    Xs, Ws = orc.scatter(X, orc.B, k), orc.scatter(W, orc.S1, k)
    got, _ = run(Xs, orc.B, Ws, orc.S1, M, kk, k * N, k, 0, 0, pitch(Xs, 0, 8, extra), pitch(Ws, 0, 8, extra), epilogue=epilogue)
    for i in range(k):
        ref = values(X) @ values(Ws[i])
        r = orc.gelu(ref) if epilogue == sbp.EPI_GELU else ref
        assert_matmul_close(got[i], r, 2.0 ** -8 + 1e-4, f"{M}x{kk}x{N} epilogue {epilogue} shard {i}")


@pytest.mark.parametrize("variant", [0, 1, 3, 4, 6, 7, 8, 9, 12, 16, 21, 40, 41, 42, 43, 44, 48])
def test_gelu_of_nan_and_infinity(variant):
    """whole steps on aligned rows, every kernel: a NaN accumulator gives NaN, +inf gives +inf, and the rows beside them do not change"""
    k, M, K, N = 2, 300, 128, 2 * 264
    X, W = bf16(50, (M, K)), bf16(51, (K, N), 0.2)
    W[0] = wl.to_bf16_bits(np.ones((1, N)))[0]
    plain, (nan, inf) = X.copy(), (13, 170)
    X[nan, 5], X[inf, 0] = 0x7FC0, 0x7F80
    Ws = orc.scatter(W, orc.S1, k)
    a, _ = run(orc.scatter(X, orc.B, k), orc.B, Ws, orc.S1, M, K, N, k, 0, 0, 0, 0, variant=variant, epilogue=sbp.EPI_GELU)
    b, _ = run(orc.scatter(plain, orc.B, k), orc.B, Ws, orc.S1, M, K, N, k, 0, 0, 0, 0, variant=variant, epilogue=sbp.EPI_GELU)
    for i in range(k):
        assert np.isnan(a[i][nan]).all(), f"v{variant}: NaN"
        assert (a[i][inf] == np.inf).all(), f"v{variant}: +inf"
        rest = np.delete(np.arange(M), [nan, inf])
        assert np.array_equal(a[i][rest], b[i][rest]), f"v{variant}: other rows"
