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
