"""Boxing and the cross-entropy gradient on rows that no 16-byte vector divides: unaligned vectors, the last one of a row
element by element.  Moves are bit-exact; reductions add in shard order, so plain fp32 sums in that order are bit-exact too."""
import numpy as np
import pytest

import oracle as orc
import paper_2110_15032_amd as sbp
import workloads as wl
from sbp_harness import DevTensor, TO_ABI, assert_bits_equal, sync

pytestmark = pytest.mark.gpu
SEED = wl.SEED_BASE + 1900
# widths: one vector and a rest on some shards, an empty rest on others, less than a vector per shard, many rows of few vectors;
# 34 columns on each of 8 and of 3 devices and 10 on each of 3: exact 8-byte vectors
SHAPES = [(5, 17), (37, 259), (130, 1031), (7, 24), (1, 8191), (600, 33), (2, 8200), (50, 272), (9, 102), (50, 30)]


def f32(tid, shape):
    return wl.normal(SEED, tid, shape).astype(np.float32)


@pytest.mark.parametrize("k,ko", [(2, 2), (3, 3), (8, 8), (3, 5)])
@pytest.mark.parametrize("words", ["u16", "f32"])
@pytest.mark.parametrize("si,so", [(orc.S0, orc.S1), (orc.S1, orc.S0), (orc.S0, orc.B), (orc.S1, orc.B), (orc.B, orc.S0), (orc.B, orc.S1), (orc.S0, orc.S0), (orc.S1, orc.S1)])
def test_moves(k, ko, words, si, so):
    for n, shape in enumerate(SHAPES):
        T = f32(n, shape) if words == "f32" else wl.to_bf16_bits(wl.normal(SEED, n, shape))
        d_in = DevTensor.from_host(orc.scatter(T, si, k), *shape, si)
        d_out = DevTensor.empty(*shape, T.dtype, so, ko)
        sbp.sbp_boxing_across(d_in.desc, TO_ABI[si], k, d_out.desc, TO_ABI[so], ko)
        sync()
        for j, (got, ref) in enumerate(zip(d_out.host(), orc.scatter(T, so, ko))):
            assert_bits_equal(got, ref, f"{si}->{so} {shape} {words} {k}->{ko} shard {j}")


@pytest.mark.parametrize("k", [1, 2, 3, 4, 5, 7, 8])
@pytest.mark.parametrize("op", ["sum", "max"])
@pytest.mark.parametrize("so", [orc.B, orc.S0, orc.S1])
def test_reductions(k, op, so):
    si = orc.P_SUM if op == "sum" else orc.P_MAX
    for n, shape in enumerate(SHAPES):
        parts = [f32(100 + 10 * n + i, shape) for i in range(k)]
        parts[0].flat[0] = -np.inf
        ref = parts[0]
        for p in parts[1:]:
            ref = ref + p if op == "sum" else np.maximum(ref, p)
        d_in = DevTensor.from_host(parts, *shape, si)
        d_out = DevTensor.empty(*shape, np.float32, so, k)
        sbp.sbp_boxing(d_in.desc, TO_ABI[si], d_out.desc, TO_ABI[so], k)
        sync()
        for j, (got, want) in enumerate(zip(d_out.host(), orc.scatter(ref, so, k))):
            assert_bits_equal(got, want, f"{op} {so} {shape} k={k} shard {j}")


@pytest.mark.parametrize("k", [2, 3, 4, 8])
@pytest.mark.parametrize("axis", [0, 1])
def test_casts(k, axis):
    sig = orc.S0 if axis == 0 else orc.S1
    for n, shape in enumerate(SHAPES):
        T = f32(200 + n, shape)
        d_in, d_out = DevTensor.from_host(orc.scatter(T, sig, k), *shape, sig), DevTensor.empty(*shape, np.uint16, orc.B, k)
        sbp.sbp_boxing_cast(d_in.desc, TO_ABI[sig], d_out.desc, sbp.B, k)
        parts = [wl.to_bf16_bits(wl.normal(SEED, 300 + 10 * n + i, shape)) for i in range(k)]
        d_p, d_s = DevTensor.from_host(parts, *shape, orc.P_SUM), DevTensor.empty(*shape, np.float32, sig, k)
        sbp.sbp_boxing_cast(d_p.desc, sbp.P_SUM, d_s.desc, TO_ABI[sig], k)
        sync()
        for j, got in enumerate(d_out.host()):
            assert_bits_equal(got, orc.bf16_round(T.astype(np.float64)), f"gather {shape} k={k} copy {j}")
        ref = np.zeros(shape, np.float32)
        for p in parts:
            ref = ref + orc.bf16_to_f64(p).astype(np.float32)
        for j, (got, want) in enumerate(zip(d_s.host(), orc.scatter(ref, sig, k))):
            assert_bits_equal(got, want, f"reduce {shape} k={k} shard {j}")


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("cols", [3, 23, 1003, 2050])
def test_cross_entropy_gradient_does_not_depend_on_the_pitch(cols, dtype):
    """dense rows (unaligned vectors) against rows padded to 16 bytes: the same bits, padding untouched; labels in the first,
    the last and the broken vector of a shard"""
    torch = __import__("torch")
    k, rows = 2, 29
    L = f32(400, (rows, cols)) * np.float32(3.0)
    if dtype == "bf16":
        L = wl.to_bf16_bits(L)
    y = (wl.uniform(SEED, 401, (rows, 1), 0.0, float(cols)).astype(np.int64) % cols).astype(np.int32)
    y[0, 0], y[1, 0], y[2, 0], y[3, 0] = 0, cols - 1, -(-cols // 2) - 1, -1
    one = lambda v: DevTensor.from_host([v] * k, rows, 1, orc.B)      # noqa: E731
    m, s, g = one(np.full((rows, 1), 2.0, np.float32)), one(np.full((rows, 1), 9.0, np.float32)), one(f32(402, (rows, 1)))
    labels = sbp.SbpTensor([torch.from_numpy(y.copy()).cuda() for _ in range(k)], rows, 1, sbp.I32)
    shards, outs = orc.scatter(L, orc.S1, k), []
    for ld in (0, -(-shards[0].shape[1] // 8) * 8):
        d_l, d_d = DevTensor.from_host(shards, rows, cols, orc.S1, ld=ld), DevTensor.empty(rows, cols, L.dtype, orc.S1, k, ld=ld)
        sbp.sbp_xent_grad(d_l.desc, sbp.S(1), labels, m.desc, s.desc, g.desc, d_d.desc, k)
        sync()
        outs.append(d_d.host())
    for i in range(k):
        assert_bits_equal(outs[0][i], outs[1][i], f"{cols} {dtype} shard {i}")


# enough elements for the vector kernels of the casts and of the gradient: rows of exactly one vector and one more, a last
# vector that shares one, three and seven elements with its neighbour, one long row
LARGE = [(40000, 9), (9000, 66), (700, 1031), (1, 600011)]


@pytest.mark.parametrize("k", [2, 3, 8])
@pytest.mark.parametrize("axis", [0, 1])
def test_casts_of_many_elements(k, axis):
    sig = orc.S0 if axis == 0 else orc.S1
    for n, shape in enumerate(LARGE):
        if axis == 1:
            shape = (shape[0], shape[1] * k) if shape[0] > 1 else shape
        T = f32(500 + n, shape)
        d_in, d_out = DevTensor.from_host(orc.scatter(T, sig, k), *shape, sig), DevTensor.empty(*shape, np.uint16, orc.B, k)
        sbp.sbp_boxing_cast(d_in.desc, TO_ABI[sig], d_out.desc, sbp.B, k)
        parts = [wl.to_bf16_bits(f32(600 + 10 * n + i, shape)) for i in range(k)]
        d_p, d_s = DevTensor.from_host(parts, *shape, orc.P_SUM), DevTensor.empty(*shape, np.float32, sig, k)
        sbp.sbp_boxing_cast(d_p.desc, sbp.P_SUM, d_s.desc, TO_ABI[sig], k)
        sync()
        want = orc.bf16_round(T.astype(np.float64))
        for j, got in enumerate(d_out.host()):
            assert_bits_equal(got, want, f"gather {shape} k={k} copy {j}")
        ref = np.zeros(shape, np.float32)
        for p in parts:
            ref = ref + orc.bf16_to_f64(p).astype(np.float32)
        for j, (got, want) in enumerate(zip(d_s.host(), orc.scatter(ref, sig, k))):
            assert_bits_equal(got, want, f"reduce {shape} k={k} shard {j}")


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("rows,cols,pad", [(70000, 16, 0), (60000, 18, 3), (9000, 67, 0), (9000, 67, 7), (600, 2050, 0), (300, 8191, 1),
                                           (60000, 18, 7), (9000, 67, 6), (300, 8191, 8)])   # the last three: aligned rows, broken last vectors
def test_cross_entropy_gradient_of_many_rows(rows, cols, pad, dtype):
    """against the same call on a few of the rows, which takes one element per lane: the same bits; padding untouched"""
    torch = __import__("torch")
    k, few = 2, 20
    L = f32(700, (rows, cols)) * np.float32(3.0)
    if dtype == "bf16":
        L = wl.to_bf16_bits(L)
    y = (np.arange(rows, dtype=np.int32) * 7 % (cols + 1) - 1).reshape(rows, 1).astype(np.int32)
    m, s, g = np.full((rows, 1), 2.0, np.float32), np.full((rows, 1), 9.0, np.float32), f32(702, (rows, 1))
    ld = -(-cols // k) + pad if pad else 0

    def grad(a, b):
        n = b - a
        one = lambda v: DevTensor.from_host([v[a:b]] * k, n, 1, orc.B).desc      # noqa: E731
        labels = sbp.SbpTensor([torch.from_numpy(y[a:b].copy()).cuda() for _ in range(k)], n, 1, sbp.I32)
        d_l, d_d = DevTensor.from_host(orc.scatter(L[a:b], orc.S1, k), n, cols, orc.S1, ld=ld), DevTensor.empty(n, cols, L.dtype, orc.S1, k, ld=ld)
        sbp.sbp_xent_grad(d_l.desc, sbp.S(1), labels, one(m), one(s), one(g), d_d.desc, k)
        sync()
        return d_d.host()

    whole = grad(0, rows)
    for a in (0, rows // 2, rows - few):
        for i, (got, want) in enumerate(zip(whole, grad(a, a + few))):
            assert_bits_equal(np.ascontiguousarray(got[a:a + few]), want, f"{rows}x{cols}+{pad} {dtype} rows from {a}, shard {i}")
