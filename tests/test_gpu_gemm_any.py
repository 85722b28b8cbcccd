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
