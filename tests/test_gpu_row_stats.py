"""Row maxima and sums of exponentials where the choice of kernel changes: few long rows (1024 threads), many (256), rows around whole
rounds of vectors, at any alignment; against numpy in float64."""
import numpy as np
import pytest

import paper_2110_15032_amd as sbp
import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bf", [True, False])
@pytest.mark.parametrize("rows,cols,k,ld", [(2, 16384, 2, 0), (3, 16383, 1, 0), (5, 33001, 3, 33007), (1, 65536 + 8, 2, 0), (600, 16391, 1, 0), (4, 4 * 8192 + 13, 2, 0), (7, 1, 2, 0), (513, 8200, 1, 8201)])
def test_row_stats(rows, cols, k, ld, bf):
    import torch
    host = wl.normal(wl.SEED_BASE + 55, rows, (rows, cols * k), 2.0).astype(np.float32)
    if bf:
        host = torch.from_numpy(host).to(torch.bfloat16).float().numpy()
    pitch = ld or cols
    parts = []
    for i in range(k):
        buf = torch.full((rows, pitch), float("nan"), dtype=torch.bfloat16 if bf else torch.float32, device="cuda")
        buf[:, :cols] = torch.from_numpy(host[:, i * cols:(i + 1) * cols]).to(buf.dtype).cuda()
        parts.append(buf)
    logits = sbp.SbpTensor(parts, rows, cols * k, sbp.BF16 if bf else sbp.F32, 0, ld)
    vec = lambda v=float("nan"): [torch.full((rows, 1), v, device="cuda") for _ in range(k)]
    top, total = vec(), vec()
    peak = torch.from_numpy(host.max(axis=1, keepdims=True)).cuda()
    sbp.sbp_row_max(logits, sbp.S(1), sbp.SbpTensor(top, rows, 1, sbp.F32), k)
    sbp.sbp_row_sumexp(logits, sbp.S(1), sbp.SbpTensor([peak] * k, rows, 1, sbp.F32), sbp.SbpTensor(total, rows, 1, sbp.F32), k)
    torch.cuda.synchronize()
    for i in range(k):
        part = host[:, i * cols:(i + 1) * cols].astype(np.float64)
        assert np.array_equal(top[i].cpu().numpy()[:, 0], part.max(axis=1).astype(np.float32))
        want = np.exp(part - peak.cpu().numpy().astype(np.float64)).sum(axis=1)
        # a term is off by 1e-7 |v - max| < 3e-6, the sum by its order: chains of at most cols / 1024 + 16 additions
        assert np.all(np.abs(total[i].cpu().numpy()[:, 0] - want) <= 1e-5 * want)


@pytest.mark.parametrize("bf", [True, False])
@pytest.mark.parametrize("rows,cols,k", [(600, 125001, 2), (1100, 20011, 7)])
def test_row_stats_streaming(rows, cols, k, bf):
    """more than 256 MiB in rows of any alignment: loads past the cache; against torch on the device"""
    import torch
    dt = torch.bfloat16 if bf else torch.float32
    pitch = cols + (5 if bf else 2)
    g = torch.Generator(device="cuda").manual_seed(wl.SEED_BASE + 56)
    parts = []
    for _ in range(k):
        buf = torch.full((rows, pitch), float("nan"), dtype=dt, device="cuda")
        buf[:, :cols].normal_(0.0, 2.0, generator=g)
        parts.append(buf)
    assert k * rows * cols * (2 if bf else 4) > 256 << 20
    logits = sbp.SbpTensor(parts, rows, cols * k, sbp.BF16 if bf else sbp.F32, 0, pitch)
    top, total = ([torch.full((rows, 1), float("nan"), device="cuda") for _ in range(k)] for _ in range(2))
    sbp.sbp_row_max(logits, sbp.S(1), sbp.SbpTensor(top, rows, 1, sbp.F32), k)
    peak = torch.stack(top).amax(0)
    sbp.sbp_row_sumexp(logits, sbp.S(1), sbp.SbpTensor([peak] * k, rows, 1, sbp.F32), sbp.SbpTensor(total, rows, 1, sbp.F32), k)
    torch.cuda.synchronize()
    for i in range(k):
        part = parts[i][:, :cols].float()
        assert torch.equal(top[i], part.amax(1, keepdim=True))
        want = torch.exp(part.double() - peak.double()).sum(1, keepdim=True)
        assert bool((torch.abs(total[i].double() - want) <= 1e-5 * want).all())


@pytest.mark.parametrize("bf", [True, False])
@pytest.mark.parametrize("rows,cols", [(4, 16391), (4, 40000), (600, 1003)])
def test_row_stats_of_nan_and_infinity(rows, cols, bf):
    """NaN next to numbers is ignored by the maximum, a row of NaN or -inf gives -inf, an infinity wins; -inf adds nothing to the sum,
    NaN shows in it; few long rows (1024 threads) and others, at the first, a middle and the last element"""
    import torch
    host = wl.normal(wl.SEED_BASE + 57, rows, (rows, cols), 2.0).astype(np.float32)
    nan, inf = np.float32("nan"), np.float32("inf")
    host[0, [0, cols // 2, cols - 1]] = nan
    host[1, :] = -inf
    host[1, cols - 1] = 0.5
    host[2, :] = -inf
    host[3, :] = nan
    plain = wl.normal(wl.SEED_BASE + 58, rows, (rows, cols), 2.0).astype(np.float32)
    plain[0, [0, cols // 3, cols - 1]] = inf
    for h in (host, plain):
        dev = torch.from_numpy(h).cuda().to(torch.bfloat16 if bf else torch.float32)
        h = dev.float().cpu().numpy()
        logits = sbp.SbpTensor([dev], rows, cols, sbp.BF16 if bf else sbp.F32)
        top, total = torch.full((rows, 1), 5.0, device="cuda"), torch.full((rows, 1), 5.0, device="cuda")
        peak = torch.full((rows, 1), 4.0, device="cuda")
        sbp.sbp_row_max(logits, sbp.S(1), sbp.SbpTensor([top], rows, 1, sbp.F32), 1)
        sbp.sbp_row_sumexp(logits, sbp.S(1), sbp.SbpTensor([peak], rows, 1, sbp.F32), sbp.SbpTensor([total], rows, 1, sbp.F32), 1)
        torch.cuda.synchronize()
        assert np.array_equal(top.cpu().numpy()[:, 0], np.fmax.reduce(h, axis=1, initial=-inf))
        want = np.exp(h.astype(np.float64) - 4.0).sum(axis=1)
        got = total.cpu().numpy()[:, 0].astype(np.float64)
        assert np.array_equal(np.isnan(got), np.isnan(want)) and np.array_equal(np.isinf(got), np.isinf(want))
        ok = np.isfinite(want)
        assert np.all(np.abs(got[ok] - want[ok]) <= 1e-5 * want[ok])
