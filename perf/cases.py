"""Performance cases of the SBP library: whole steps of the programs it is written for, through its public entry points.

A case is a dict of plain values.  `kind` names the program, `k` the number of logical devices (shard buffers in one
GPU's memory); the other entries are global sizes.  Every kind covers a range of sizes, from single tokens and tens of
rows to the workloads of `workloads/configs.py` and `bench.py`, with lengths that are multiples of 128, multiples of 8
and odd:

  f32         X S(1) x W S(0) -> P(sum) in fp32, boxed to B and to S(0)                      (`tiny` of the workloads)
  mlp         gelu(X W1) W2 -> P(sum) -> B, column- then row-parallel; grid > 1: the same product chain (without the
              activation) on a grid x k device grid, data-parallel outside and model-parallel inside
  mlp_bwd     the gradients of that block: dH = dY W2^T, dW2 = H^T dY, dW1 = X^T dA, dX = dA W1^T -> P(sum) -> B
  dp_grad     dW = X^T dY over token shards -> P(sum), boxed to S(0) and to B
  classifier  training step of the model-parallel head: logits with the local row maxima, softmax statistics, sparse
              cross entropy, gradient of the logits, gradients of the features (P(sum) -> B) and of the weight
  uvw         U V W with deferred boxing: the fp32 partials of U V meet a bf16 W, one P(sum) -> B at the end
  relayout    S(0) -> S(1) -> B -> S(0) on k devices, then S(0) over to k_out other devices (raw words)
  zero        sharded optimizer state: fp32 S(0) -> bf16 B and bf16 P(sum) -> fp32 S(0)
"""
import math

import torch

import paper_2110_15032_amd as sbp

TORCH = {sbp.F32: torch.float32, sbp.BF16: torch.bfloat16}
BYTES = {sbp.F32: 4, sbp.BF16: 2}


def listed():
    return [
        # the smallest product and its two reductions: launch and latency bound
        dict(name="f32 tiny", kind="f32", k=2, M=64, K=128, N=96),
        # fp32 training without mixed precision, ordinary layer sizes that divide nothing evenly
        dict(name="f32 layer", kind="f32", k=4, M=2000, K=3000, N=1500),
        # Megatron-style MLP block at its full size: the headline workload
        dict(name="mlp 8192 tokens", kind="mlp", k=8, grid=1, T=8192, D=4096, F=16384),
        # the same block in decoding: a batch of single tokens, the weights are the traffic
        dict(name="mlp 32 tokens", kind="mlp", k=8, grid=1, T=32, D=4096, F=16384),
        # a last, uneven batch through a layer whose widths are multiples of 8 only
        dict(name="mlp ragged", kind="mlp", k=3, grid=1, T=777, D=1000, F=3000),
        # backward of an ordinary block on four devices
        dict(name="mlp backward", kind="mlp_bwd", k=4, T=2048, D=2048, F=8192),
        # data-parallel weight gradient at its full size
        dict(name="dp gradient", kind="dp_grad", k=8, T=16384, D=1024, F=4096),
        # face-recognition head, a million classes: the largest training step
        dict(name="classifier 1M", kind="classifier", k=8, R=1024, D=512, C=1000000, f32=False, pad=True),
        # a small head on an odd number of classes, rows back to back
        dict(name="classifier odd", kind="classifier", k=4, R=200, D=256, C=30011, f32=False, pad=False),
        # deferred boxing, sizes of the benchmark
        dict(name="uvw", kind="uvw", k=8, M=4096, K=16384, N=4096, P=1024),
        # relayout of 1 GiB on 16 devices and the hand-over to the next stage's four
        dict(name="relayout 1 GiB", kind="relayout", k=16, k_out=4, R=65536, C=8192, f32=False),
        # sharded optimizer state of 2^28 parameters
        dict(name="zero 2^28", kind="zero", k=8, R=16384, C=16384),
    ]


def _size(rng, lo, hi, step):
    """Spread over the logarithm of lo .. hi, a multiple of step."""
    n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    return max(step, (n + step // 2) // step * step)


def draw(rng):
    kind = rng.choice(["f32", "mlp", "mlp", "mlp_bwd", "dp_grad", "classifier", "classifier", "uvw", "relayout", "zero"])
    k = rng.choice([2, 3, 4, 8])
    step = rng.choice([1, 8, 128, 128])           # of the widths; token and row counts are what they are
    big = step == 128
    if kind == "f32":
        return dict(kind=kind, k=k, M=_size(rng, 32, 3000, 1), K=_size(rng, 64, 4000, min(step, 8)), N=_size(rng, 32, 3000, min(step, 8)))
    if kind == "mlp":
        D = _size(rng, 256, 4096 if big else 2048, step)
        return dict(kind=kind, k=k, grid=rng.choice([1, 1, 2]), T=_size(rng, 2, 8192 if big else 2048, 1), D=D, F=min(16384, 4 * D) if big else _size(rng, 1000, 8192, step))
    if kind == "mlp_bwd":
        D = _size(rng, 256, 2048, step)
        return dict(kind=kind, k=k, T=_size(rng, 16, 4096 if big else 2048, 1), D=D, F=4 * D if big else _size(rng, 1000, 6000, step))
    if kind == "dp_grad":
        return dict(kind=kind, k=k, T=_size(rng, 256, 16384, step), D=_size(rng, 128, 1024, step), F=_size(rng, 512, 4096, step))
    if kind == "classifier":
        f32 = rng.random() < 0.25
        return dict(kind=kind, k=k, R=_size(rng, 8, 1024, 1), D=_size(rng, 64, 512, max(8, min(step, 64))), C=_size(rng, 1000, 50000 if f32 else 500000, step), f32=f32, pad=rng.random() < 0.5)
    if kind == "uvw":
        return dict(kind=kind, k=k, M=_size(rng, 64, 4096 if big else 1024, 1), K=_size(rng, 512, 16384 if big else 4096, step), N=_size(rng, 256, 4096 if big else 1024, step),
                    P=_size(rng, 64, 1024, step))
    if kind == "relayout":
        return dict(kind=kind, k=rng.choice([2, 3, 4, 8, 16]), k_out=rng.choice([2, 4, 5]), R=_size(rng, 64, 65536, 1), C=_size(rng, 64, 4096, step), f32=rng.random() < 0.5)
    return dict(kind=kind, k=k, R=_size(rng, 64, 16384, 1), C=_size(rng, 64, 8192, step))


# ---------------------------------------------------------------------------------------------------------------------
# tensors: k local buffers and the descriptor that the library takes
# ---------------------------------------------------------------------------------------------------------------------
class _Maker:
    def __init__(self, seed):
        self.gen = torch.Generator(device="cuda")
        self.gen.manual_seed(seed)

    def _normal(self, shape, dtype, std):
        t = torch.empty(shape, dtype=TORCH[dtype], device="cuda")
        return t.normal_(0.0, std, generator=self.gen)

    @staticmethod
    def _shapes(rows, cols, sig, k, grid):
        if grid == 1:
            return [sbp.sbp_local_shape(rows, cols, sig, k, i) for i in range(k)]
        return [sbp.sbp_local_shape_2d(rows, cols, sig, grid, k, a, b) for a in range(grid) for b in range(k)]

    def normal(self, rows, cols, sig, k, dtype, std=1.0, trans=0, grid=1):
        """An input of N(0, std^2) values; the devices of a B input hold copies of their own."""
        shapes = [(c, r) if trans else (r, c) for r, c in self._shapes(rows, cols, sig, k, grid)]
        if sig == sbp.B:
            one = self._normal(shapes[0], dtype, std)
            parts = [one] + [one.clone() for _ in range(k - 1)]
        else:
            parts = [self._normal(s, dtype, std) for s in shapes]
            if grid > 1:      # devices that hold the same slice hold the same values
                for a in range(grid):
                    for b in range(k):
                        src = (0 if sig[0] == sbp.B else a) * k + (0 if sig[1] == sbp.B else b)
                        parts[a * k + b].copy_(parts[src])
        return sbp.SbpTensor(parts, rows, cols, dtype, trans)

    def empty(self, rows, cols, sig, k, dtype, grid=1):
        parts = [torch.zeros(s, dtype=TORCH[dtype], device="cuda") for s in self._shapes(rows, cols, sig, k, grid)]
        return sbp.SbpTensor(parts, rows, cols, dtype)

    def pitched(self, rows, cols, k, dtype):
        """An S(1) output whose rows start on cache lines (128 bytes)."""
        line = 128 // BYTES[dtype]
        ld = (-(-cols // k) + line - 1) // line * line
        parts = [torch.zeros((rows, ld), dtype=TORCH[dtype], device="cuda") for _ in range(k)]
        return sbp.SbpTensor(parts, rows, cols, dtype, 0, ld)

    def words(self, rows, cols, sig, k, dtype):
        whole = {sbp.F32: torch.int32, sbp.BF16: torch.int16}[dtype]
        info = torch.iinfo(whole)
        parts = [torch.randint(info.min, info.max, s, dtype=whole, device="cuda", generator=self.gen) for s in self._shapes(rows, cols, sig, k, 1)]
        return sbp.SbpTensor(parts, rows, cols, dtype)

    def no_words(self, rows, cols, sig, k, dtype):
        whole = {sbp.F32: torch.int32, sbp.BF16: torch.int16}[dtype]
        parts = [torch.zeros(s, dtype=whole, device="cuda") for s in self._shapes(rows, cols, sig, k, 1)]
        return sbp.SbpTensor(parts, rows, cols, dtype)


S0, S1, B, PS, PM = sbp.S(0), sbp.S(1), sbp.B, sbp.P_SUM, sbp.P_MAX
F32, BF16 = sbp.F32, sbp.BF16


def prepare(case, seed):
    m = _Maker(seed)
    kind, k = case["kind"], case["k"]
    s = dict(case=case)
    if kind == "f32":
        M, K, N = case["M"], case["K"], case["N"]
        s.update(X=m.normal(M, K, S1, k, F32), W=m.normal(K, N, S0, k, F32, 0.1), Y=m.empty(M, N, PS, k, F32), YB=m.empty(M, N, B, k, F32), YS=m.empty(M, N, S0, k, F32))
    elif kind == "mlp":
        T, D, F, g = case["T"], case["D"], case["F"], case["grid"]
        if g == 1:
            s.update(X=m.normal(T, D, B, k, BF16), W1=m.normal(D, F, S1, k, BF16, 0.02), W2=m.normal(F, D, S0, k, BF16, 0.02), H=m.empty(T, F, S1, k, BF16),
                     Y=m.empty(T, D, PS, k, F32), YB=m.empty(T, D, B, k, F32))
        else:
            s.update(X=m.normal(T, D, (S0, B), k, BF16, 1.0, 0, g), W1=m.normal(D, F, (B, S1), k, BF16, 0.02, 0, g), W2=m.normal(F, D, (B, S0), k, BF16, 0.02, 0, g),
                     H=m.empty(T, F, (S0, S1), k, BF16, g), Y=m.empty(T, D, (S0, PS), k, F32, g), YB=m.empty(T, D, (S0, B), k, F32, g))
    elif kind == "mlp_bwd":
        T, D, F = case["T"], case["D"], case["F"]
        X, H = m.normal(T, D, B, k, BF16), m.normal(T, F, S1, k, BF16)
        W1, W2 = m.normal(D, F, S1, k, BF16, 0.02), m.normal(F, D, S0, k, BF16, 0.02)
        dA = m.normal(T, F, S1, k, BF16, 0.05)     # gradient of the pre-activations
        s.update(dY=m.normal(T, D, B, k, BF16), dA=dA, keep=(X, H, W1, W2),
                 XT=sbp.SbpTensor(X.keep, D, T, BF16, 1), HT=sbp.SbpTensor(H.keep, F, T, BF16, 1), W1T=sbp.SbpTensor(W1.keep, F, D, BF16, 1), W2T=sbp.SbpTensor(W2.keep, D, F, BF16, 1),
                 dH=m.empty(T, F, S1, k, BF16), dW2=m.empty(F, D, S0, k, BF16), dW1=m.empty(D, F, S1, k, BF16), dX=m.empty(T, D, PS, k, F32), dXB=m.empty(T, D, B, k, F32))
    elif kind == "dp_grad":
        T, D, F = case["T"], case["D"], case["F"]
        s.update(XT=m.normal(D, T, S1, k, BF16, 1.0, 1), dY=m.normal(T, F, S0, k, BF16), dW=m.empty(D, F, PS, k, F32), dWS=m.empty(D, F, S0, k, F32), dWB=m.empty(D, F, B, k, F32))
    elif kind == "classifier":
        R, D, C, dt = case["R"], case["D"], case["C"], F32 if case["f32"] else BF16
        F, W = m.normal(R, D, B, k, dt), m.normal(D, C, S1, k, dt, 0.01)
        logits = (lambda: m.pitched(R, C, k, dt)) if case["pad"] else (lambda: m.empty(R, C, S1, k, dt))
        labels = torch.randint(0, C, (R, 1), dtype=torch.int32, device="cuda", generator=m.gen)
        grad = torch.full((R, 1), 1.0 / R, device="cuda")
        s.update(F=F, W=W, L=logits(), dL=logits(), labels=sbp.SbpTensor([labels] * k, R, 1, sbp.I32), grad=sbp.SbpTensor([grad] * k, R, 1, F32),
                 FT=sbp.SbpTensor(F.keep, D, R, dt, 1), WT=sbp.SbpTensor(W.keep, C, D, dt, 1),
                 dF=m.empty(R, D, PS, k, F32), dFB=m.empty(R, D, B, k, F32), dW=m.empty(D, C, S1, k, dt))
        s.update((v, m.empty(R, 1, B, k, F32)) for v in ("maxP", "maxB", "sumP", "sumB", "lossP", "lossB"))
    elif kind == "uvw":
        M, K, N, P = case["M"], case["K"], case["N"], case["P"]
        s.update(U=m.normal(M, K, S1, k, BF16), V=m.normal(K, N, S0, k, BF16, 0.02), W=m.normal(N, P, B, k, BF16, 0.02), UV=m.empty(M, N, PS, k, F32), Y=m.empty(M, P, PS, k, F32),
                 YB=m.empty(M, P, B, k, F32))
    elif kind == "relayout":
        R, C, dt, ko = case["R"], case["C"], F32 if case["f32"] else BF16, case["k_out"]
        s.update(T0=m.words(R, C, S0, k, dt), T1=m.no_words(R, C, S1, k, dt), TB=m.no_words(R, C, B, k, dt), T2=m.no_words(R, C, S0, k, dt), TO=m.no_words(R, C, S0, ko, dt))
    else:
        R, C = case["R"], case["C"]
        s.update(W32=m.normal(R, C, S0, k, F32, 0.02), W16=m.empty(R, C, B, k, BF16), G16=m.normal(R, C, PS, k, BF16), G32=m.empty(R, C, S0, k, F32))
    return s


def run(s):
    c = s["case"]
    kind, k = c["kind"], c["k"]
    if kind == "f32":
        sbp.sbp_matmul(s["X"], S1, s["W"], S0, s["Y"], PS, k)
        sbp.sbp_boxing(s["Y"], PS, s["YB"], B, k)
        sbp.sbp_boxing(s["Y"], PS, s["YS"], S0, k)
        return [s[v].keep for v in ("Y", "YB", "YS")]
    if kind == "mlp":
        g = c["grid"]
        if g == 1:
            sbp.sbp_matmul_ex(s["X"], B, s["W1"], S1, s["H"], S1, k, None, sbp.EPI_GELU)
            sbp.sbp_matmul(s["H"], S1, s["W2"], S0, s["Y"], PS, k)
            sbp.sbp_boxing(s["Y"], PS, s["YB"], B, k)
        else:
            sbp.sbp_matmul_2d(s["X"], (S0, B), s["W1"], (B, S1), s["H"], (S0, S1), g, k)
            sbp.sbp_matmul_2d(s["H"], (S0, S1), s["W2"], (B, S0), s["Y"], (S0, PS), g, k)
            sbp.sbp_boxing_2d(s["Y"], (S0, PS), s["YB"], (S0, B), g, k)
        return [s[v].keep for v in ("H", "Y", "YB")]
    if kind == "mlp_bwd":
        sbp.sbp_matmul(s["dY"], B, s["W2T"], S1, s["dH"], S1, k)
        sbp.sbp_matmul(s["HT"], S0, s["dY"], B, s["dW2"], S0, k)
        sbp.sbp_matmul(s["XT"], B, s["dA"], S1, s["dW1"], S1, k)
        sbp.sbp_matmul(s["dA"], S1, s["W1T"], S0, s["dX"], PS, k)
        sbp.sbp_boxing(s["dX"], PS, s["dXB"], B, k)
        return [s[v].keep for v in ("dH", "dW2", "dW1", "dX", "dXB")]
    if kind == "dp_grad":
        sbp.sbp_matmul(s["XT"], S1, s["dY"], S0, s["dW"], PS, k)
        sbp.sbp_boxing(s["dW"], PS, s["dWS"], S0, k)
        sbp.sbp_boxing(s["dW"], PS, s["dWB"], B, k)
        return [s[v].keep for v in ("dW", "dWS", "dWB")]
    if kind == "classifier":
        L, dL = s["L"], s["dL"]
        sbp.sbp_matmul_rowmax(s["F"], B, s["W"], S1, L, S1, s["maxP"], k)
        sbp.sbp_boxing(s["maxP"], PM, s["maxB"], B, k)
        sbp.sbp_row_sumexp(L, S1, s["maxB"], s["sumP"], k)
        sbp.sbp_boxing(s["sumP"], PS, s["sumB"], B, k)
        sbp.sbp_xent_loss(L, S1, s["labels"], s["maxB"], s["sumB"], s["lossP"], k)
        sbp.sbp_boxing(s["lossP"], PS, s["lossB"], B, k)
        sbp.sbp_xent_grad(L, S1, s["labels"], s["maxB"], s["sumB"], s["grad"], dL, k)
        sbp.sbp_matmul(dL, S1, s["WT"], S0, s["dF"], PS, k)
        sbp.sbp_boxing(s["dF"], PS, s["dFB"], B, k)
        sbp.sbp_matmul(s["FT"], B, dL, S1, s["dW"], S1, k)
        cols = [c["C"] // k + (i < c["C"] % k) for i in range(k)]
        return [[t[:, :n] for t, n in zip(v.keep, cols)] for v in (L, dL)] + [s[v].keep for v in ("maxB", "sumB", "lossB", "dF", "dFB", "dW")]
    if kind == "uvw":
        sbp.sbp_matmul(s["U"], S1, s["V"], S0, s["UV"], PS, k)
        sbp.sbp_matmul(s["UV"], PS, s["W"], B, s["Y"], PS, k)
        sbp.sbp_boxing(s["Y"], PS, s["YB"], B, k)
        return [s[v].keep for v in ("UV", "Y", "YB")]
    if kind == "relayout":
        sbp.sbp_boxing(s["T0"], S0, s["T1"], S1, k)
        sbp.sbp_boxing(s["T1"], S1, s["TB"], B, k)
        sbp.sbp_boxing(s["TB"], B, s["T2"], S0, k)
        sbp.sbp_boxing_across(s["T2"], S0, k, s["TO"], S0, c["k_out"])
        return [s[v].keep for v in ("T1", "TB", "T2", "TO")]
    sbp.sbp_boxing_cast(s["W32"], S0, s["W16"], B, k)
    sbp.sbp_boxing_cast(s["G16"], PS, s["G32"], S0, k)
    return [s[v].keep for v in ("W16", "G32")]


def work(case):
    """Every call reads each of its input buffers once and writes each of its output buffers once."""
    kind, k = case["kind"], case["k"]
    if kind == "f32":
        M, K, N = case["M"], case["K"], case["N"]
        return dict(flops=2 * M * K * N, bytes=4 * (M * K + K * N + k * M * N + 2 * k * M * N + (k + 1) * M * N))
    if kind == "mlp":
        T, D, F, g = case["T"], case["D"], case["F"], case["grid"]
        return dict(flops=4 * T * D * F, bytes=2 * (k * T * D + g * 2 * D * F + 2 * T * F) + 4 * 3 * k * T * D)
    if kind == "mlp_bwd":
        T, D, F = case["T"], case["D"], case["F"]
        return dict(flops=8 * T * D * F, bytes=2 * (2 * k * T * D + k * T * D + 4 * T * F + 4 * D * F) + 4 * 3 * k * T * D)
    if kind == "dp_grad":
        T, D, F = case["T"], case["D"], case["F"]
        return dict(flops=2 * T * D * F, bytes=2 * T * (D + F) + 4 * D * F * (k + k + 1 + 2 * k))
    if kind == "classifier":
        R, D, C, e = case["R"], case["D"], case["C"], 4 if case["f32"] else 2
        return dict(flops=6 * R * D * C, bytes=e * (2 * k * R * D + 3 * D * C + 6 * R * C) + 4 * 3 * k * R * D)
    if kind == "uvw":
        M, K, N, P = case["M"], case["K"], case["N"], case["P"]
        return dict(flops=2 * M * K * N + 2 * k * M * N * P, bytes=2 * (M * K + K * N + k * N * P) + 4 * k * (2 * M * N + 3 * M * P))
    if kind == "relayout":
        return dict(flops=0, bytes=(4 if case["f32"] else 2) * case["R"] * case["C"] * (2 + 1 + k + 2 + 2))
    return dict(flops=0, bytes=case["R"] * case["C"] * (4 + 2 * k + 2 * k + 4))


def tolerance(case):
    """Four times what the same products show with their sums in another order, or against 64 bits."""
    if case["kind"] in ("relayout", "zero"):   # words are moved, single values rounded, sums taken in shard order: one result
        return "exact"
    if case["kind"] in ("f32", "dp_grad", "uvw") or case.get("f32"):
        # fp32 sums: 5e-7 and 4e-6 (largest) over 750 terms, 7e-7 and 5e-6 over 4096, growing with the root of the length
        return dict(rel=1e-5, max=1e-4)
    # bf16 results: single values fall on the other side of a rounding, 1.1e-4 in all, one step of 2^-7 the largest
    return dict(rel=5e-4, max=0.04)
