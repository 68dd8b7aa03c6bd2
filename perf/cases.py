"""Timed work of the sketched product: what a program that uses this package has it do.

Every case goes through the package's public entry points with the buffers
such a program keeps (workspace, output, plan).  Kinds of case:

  matmul       ``matmul`` (FP32 operands, B row-major or column-major, every
               precision of the block product) with a host keep-mask
  cmask        ``matmul_cmask``: a keep mask per b x b block of C
  staged       ``sketch_cols``, ``sketch_rows`` and ``gemm_kept`` with a
               prepared sketch that is kept between calls
  weight_grad  ``autograd.sketched_weight_grad``: dW = X^T dY of a linear
               layer, sketched over the tokens
  gram         ``GramBatch.run``: a batch of sketched Hessians A D A^T

``exact`` computes the same outputs in 64 bits from the definition (SplitMix64
buckets and signs, index sums, dense products) with torch alone.
"""
import math
import random

import numpy as np
import torch

import paper_1811_02653_amd as osk
from paper_1811_02653_amd.autograd import sketched_weight_grad

DEV = "cuda"


def listed():
    return [
        # the smallest call: a product whose time is launches and latency
        dict(name="smallest_fp32", kind="matmul", m=128, n=2048, l=96, b=128, N=4, e=1, drop=1,
             precision="fp32", b_cols=False, data="iid"),
        # the small validation product (one 256 x 256 tile of C)
        dict(name="small_fp32", kind="matmul", m=256, n=4096, l=256, b=256, N=4, e=1, drop=1,
             precision="fp32", b_cols=False, data="iid"),
        # an ordinary product with no size a multiple of anything
        dict(name="ragged_fp32", kind="matmul", m=3333, n=20011, l=2777, b=900, N=4, e=1, drop=1,
             precision="fp32", b_cols=False, data="lowrank"),
        # the benchmark's workload: the large FP32 product, and its BF16 and FP8 forms
        dict(name="large_fp32", kind="matmul", m=8192, n=32768, l=8192, b=1024, N=8, e=2, drop=2,
             precision="fp32", b_cols=False, data="lowrank"),
        dict(name="large_bf16", kind="matmul", m=8192, n=32768, l=8192, b=1024, N=8, e=2, drop=2,
             precision="bf16", b_cols=False, data="lowrank"),
        dict(name="large_fp8", kind="matmul", m=8192, n=32768, l=8192, b=1024, N=8, e=2, drop=2,
             precision="fp8", b_cols=False, data="lowrank"),
        # ordinary sizes in the split precisions (log-normal row and column norms)
        dict(name="mid_bf16x3", kind="matmul", m=4096, n=16384, l=4096, b=1024, N=4, e=1, drop=1,
             precision="bf16x3", b_cols=False, data="lognormal"),
        dict(name="mid_fp8x3", kind="matmul", m=2048, n=8192, l=2048, b=512, N=4, e=1, drop=1,
             precision="fp8x3", b_cols=True, data="lognormal"),
        # stragglers per block of C, B = A^T (the paper's layout at m = 10 b, n = 60 b, z = 30 b)
        dict(name="stragglers_cmask", kind="cmask", m=5120, n=30720, l=5120, b=512, N=26, e=4,
             drop=4),
        # the steps called one by one, one prepared sketch for many products
        dict(name="staged_fp32", kind="staged", m=2048, n=16384, l=1536, b=512, N=8, e=2, drop=2),
        # the weight gradient of a linear layer in BF16
        dict(name="weight_grad_bf16", kind="weight_grad", tokens=16384, d_in=4096, d_out=4096,
             b=512, N=4, e=0, dtype="bfloat16", precision="bf16"),
        # sketched Hessians of an interior-point method, sizes spread as in the benchmark's batch
        dict(name="hessian_batch", kind="gram", count=8, m_lo=500, m_hi=4000, ratio=20, sizes=5,
             N=6, e=1, drop=1),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _side(rng, lo, hi):
    """A size over the range of lo .. hi, half of them multiples of 64."""
    x = _log_int(rng, lo, hi)
    return max(lo, x // 64 * 64) if rng.random() < 0.5 else x


def draw(rng):
    kind = rng.choices(["matmul", "cmask", "staged", "weight_grad", "gram"], [6, 1, 2, 2, 1])[0]
    if kind == "matmul":
        return dict(kind=kind, m=_side(rng, 96, 8192), n=_side(rng, 2048, 32768),
                    l=_side(rng, 96, 8192), b=_side(rng, 128, 1024), N=rng.randint(2, 7),
                    e=rng.randint(1, 2), drop=1,
                    precision=rng.choice(["fp32", "fp32", "fp32", "bf16", "bf16x3", "fp8", "fp8x3"]),
                    b_cols=rng.random() < 0.3, data=rng.choice(["iid", "lowrank", "lognormal"]))
    if kind == "cmask":
        b = rng.choice([128, 200, 256, 384, 500, 512])
        t = rng.randint(2, 10)
        return dict(kind=kind, m=t * b, n=rng.randint(10, 60) * b, l=t * b, b=b,
                    N=rng.randint(6, 20), e=4, drop=rng.randint(1, 4))
    if kind == "staged":
        return dict(kind=kind, m=_side(rng, 256, 4096), n=_side(rng, 2048, 32768),
                    l=_side(rng, 256, 4096), b=_side(rng, 128, 1024), N=rng.randint(2, 8), e=2,
                    drop=rng.randint(1, 2))
    if kind == "weight_grad":
        return dict(kind=kind, tokens=_side(rng, 2048, 16384), d_in=_side(rng, 256, 4096),
                    d_out=_side(rng, 256, 4096), b=_side(rng, 128, 512), N=rng.randint(2, 4), e=0,
                    dtype=rng.choice(["bfloat16", "bfloat16", "float32"]),
                    precision=rng.choice(["bf16", "fp32"]))
    return dict(kind=kind, count=rng.randint(2, 6), m_lo=500, m_hi=rng.randint(800, 3500), ratio=20,
                sizes=rng.randint(0, 1 << 20), N=6, e=1, drop=1)


# ---- inputs -----------------------------------------------------------------
def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed) * 1000003 + 7)


def _randn(g, *shape):
    return torch.randn(shape, generator=g, device=DEV, dtype=torch.float32)


def _pair(case, g):
    """A (m x n) and B (n x l), row-major."""
    m, n, l = case["m"], case["n"], case["l"]
    A, B = _randn(g, m, n), _randn(g, n, l)
    if case.get("data") == "lowrank":        # factors shared by A and B, and noise
        Q = _randn(g, 64, n)
        A = torch.addmm(A, _randn(g, m, 64), Q, beta=0.1, alpha=0.125)
        B = torch.addmm(B, Q.t(), _randn(g, 64, l), beta=0.1, alpha=0.125)
    elif case.get("data") == "lognormal":    # row norms of A, column norms of B
        A *= torch.exp(2 * _randn(g, m, 1)) / math.sqrt(n)
        B *= torch.exp(2 * _randn(g, 1, l)) / math.sqrt(n)
    return A, B


def _keep(case, seed, count=1):
    """count host masks over the N + e blocks, `drop` of them dropped in each."""
    total = case["N"] + case["e"]
    rng = random.Random(int(seed) * 7919 + 11)
    masks = []
    for _ in range(count):
        mask = np.ones(total, dtype=np.uint8)
        mask[rng.sample(range(total), case["drop"])] = 0
        masks.append(mask)
    return masks


def _cmask(case, seed):
    t = -(-case["m"] // case["b"])
    u = -(-case["l"] // case["b"])
    return np.stack(_keep(case, seed, t * u)).reshape(t, u, -1)


def _hessian_sizes(case):
    rng = random.Random(case["sizes"])
    return [rng.randint(case["m_lo"], case["m_hi"]) for _ in range(case["count"])]


def _hessian_inputs(case, seed):
    g = _gen(seed)
    As, ds = [], []
    for m in _hessian_sizes(case):
        n = case["ratio"] * m
        As.append(_randn(g, m, n))
        ds.append(torch.exp(torch.empty(n, device=DEV).uniform_(math.log(1e-6), math.log(1e6),
                                                                generator=g)))
    return As, ds


def _layer_inputs(case, seed):
    g = _gen(seed)
    dtype = getattr(torch, case["dtype"])
    return (_randn(g, case["tokens"], case["d_in"]).to(dtype),
            _randn(g, case["tokens"], case["d_out"]).to(dtype))


def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case, "seed": seed}
    if kind == "gram":
        As, ds = _hessian_inputs(case, seed)
        sizes = _hessian_sizes(case)
        s["plan"] = osk.GramBatch(As, ds, b=[(m + 1) // 2 for m in sizes], N=case["N"], e=case["e"],
                                  seeds=[seed + k for k in range(len(sizes))],
                                  keeps=_keep(case, seed, len(sizes)))
        return s
    b, N, e = case["b"], case["N"], case["e"]
    if kind == "weight_grad":
        s["X"], s["dY"] = _layer_inputs(case, seed)
        return s
    m, n, l = case["m"], case["n"], case["l"]
    g = _gen(seed)
    if kind == "cmask":
        s["A"] = _randn(g, m, n)
        s["B"] = s["A"].t() if m == l else _randn(g, l, n).t()
        s["cmask"] = torch.from_numpy(_cmask(case, seed)).to(DEV)
        s["workspace"] = torch.empty(osk.workspace_bytes(m, n, l, b, N, e, True), dtype=torch.uint8,
                                     device=DEV)
        s["out"] = torch.empty(m, l, device=DEV)
        return s
    s["A"], s["B"] = _pair(case, g)
    s["keep"] = _keep(case, seed)[0]
    s["out"] = torch.empty(m, l, device=DEV)
    if kind == "matmul":
        if case["b_cols"]:
            s["B"] = s["B"].t().contiguous().t()
        s["workspace"] = torch.empty(osk.workspace_bytes(m, n, l, b, N, e, case["b_cols"],
                                                         case["precision"]),
                                     dtype=torch.uint8, device=DEV)
        return s
    w = (N + e) * osk.block_stride(b)
    s["prep"] = osk.sketch_prepare(n, b, N, e, seed=seed)
    s["At"] = torch.empty(m, w, device=DEV)
    s["Bt"] = torch.empty(l, w, device=DEV)
    s["workspace"] = torch.empty(osk.sketch_rows_workspace_bytes(n, l), dtype=torch.uint8,
                                 device=DEV)
    return s


def run(s):
    case, seed = s["case"], s["seed"]
    kind = case["kind"]
    if kind == "gram":
        return s["plan"].run()
    b, N, e = case["b"], case["N"], case["e"]
    if kind == "weight_grad":
        return sketched_weight_grad(s["X"], s["dY"], b, N, e, seed=seed,
                                    precision=case["precision"])
    if kind == "cmask":
        return osk.matmul_cmask(s["A"], s["B"], b, N, e, s["cmask"], seed=seed, out=s["out"],
                                workspace=s["workspace"])
    if kind == "matmul":
        return osk.matmul(s["A"], s["B"], b, N, e, seed=seed, keep=s["keep"], out=s["out"],
                          workspace=s["workspace"], precision=case["precision"])
    At = osk.sketch_cols(s["A"], b, N, e, seed=seed, prep=s["prep"], out=s["At"])
    Bt = osk.sketch_rows(s["B"], b, N, e, seed=seed, prep=s["prep"], out=s["Bt"],
                         workspace=s["workspace"])
    return At, Bt, osk.gemm_kept(At, Bt, b, keep=s["keep"], out=s["out"])


# ---- what one pass cannot do without ----------------------------------------
def work(case):
    kind = case["kind"]
    if kind == "gram":
        nbytes = flops = 0
        for m in _hessian_sizes(case):
            n, b, K = case["ratio"] * m, (m + 1) // 2, case["N"] + case["e"] - case["drop"]
            nbytes += 4 * (m * n + n + m * m)
            flops += m * (m + 1) * K * b + 2 * K * m * n      # the upper triangle; the sketch
        return {"bytes": nbytes, "flops": flops}
    if kind == "weight_grad":
        t, p, q = case["tokens"], case["d_in"], case["d_out"]
        size = 2 if case["dtype"] == "bfloat16" else 4
        return {"bytes": size * t * (p + q) + 4 * p * q,
                "flops": 2 * p * q * case["N"] * case["b"] + 2 * case["N"] * t * (p + q)}
    m, n, l, b = case["m"], case["n"], case["l"], case["b"]
    K = case["N"] + case["e"] - case["drop"]
    T = case["N"] + case["e"]
    if kind == "cmask":
        read = m * n + (0 if m == l else n * l)
        return {"bytes": 4 * (read + m * l), "flops": 2 * m * l * K * b + 2 * T * n * (m + l)}
    nbytes = 4 * (m * n + n * l + m * l)
    if kind == "staged":
        nbytes += 4 * (m + l) * T * b
        return {"bytes": nbytes, "flops": 2 * m * l * K * b + 2 * T * n * (m + l)}
    return {"bytes": nbytes, "flops": 2 * m * l * K * b + 2 * K * n * (m + l)}


# ---- the same outputs in 64 bits --------------------------------------------
def _hash(seed, i, n, b):
    """Buckets and signs of block i (SplitMix64 at (i << 40) | k)."""
    with np.errstate(over="ignore"):
        k = np.arange(n, dtype=np.uint64) | (np.uint64(i) << np.uint64(40))
        w = np.uint64(int(seed) & (2**64 - 1)) + (k + np.uint64(1)) * np.uint64(0x9E3779B97F4A7C15)
        w = (w ^ (w >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
        w = (w ^ (w >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
        w = w ^ (w >> np.uint64(31))
    h = ((w >> np.uint64(32)) * np.uint64(b)) >> np.uint64(32)
    sign = 1.0 - 2.0 * (w & np.uint64(1)).astype(np.float64)
    return (torch.from_numpy(h.astype(np.int64)).to(DEV), torch.from_numpy(sign).to(DEV))


def _sketch64(X, seed, i, b):
    """X S_i for X with the sketched dimension last, in 64 bits."""
    h, sign = _hash(seed, i, X.shape[1], b)
    out = torch.zeros(X.shape[0], b, dtype=torch.float64, device=DEV)
    step = max(1, (1 << 28) // X.shape[1])
    for r in range(0, X.shape[0], step):
        out[r:r + step].index_add_(1, h, X[r:r + step].double() * sign)
    return out


def exact(case, seed):
    kind = case["kind"]
    if kind == "gram":
        As, ds = _hessian_inputs(case, seed)
        masks = _keep(case, seed, len(As))
        out = []
        for k, (A, d) in enumerate(zip(As, ds)):
            b = (A.shape[0] + 1) // 2
            kept = [i for i in range(len(masks[k])) if masks[k][i]]
            H = torch.zeros(A.shape[0], A.shape[0], dtype=torch.float64, device=DEV)
            W = A.double() * d.double().sqrt()
            for i in kept:
                Y = _sketch64(W, seed + k, i, b)
                H += Y @ Y.t()
            out.append(H / len(kept))
        return out
    b, N, e = case["b"], case["N"], case["e"]
    if kind == "weight_grad":
        X, dY = _layer_inputs(case, seed)
        C = 0
        for i in range(N):
            C = C + _sketch64(X.t(), seed, i, b) @ _sketch64(dY.t(), seed, i, b).t()
        return C / N
    m, l = case["m"], case["l"]
    g = _gen(seed)
    if kind == "cmask":
        A = _randn(g, m, case["n"])
        Bt = A if m == l else _randn(g, l, case["n"])
        mask = torch.from_numpy(_cmask(case, seed)).to(DEV).double()
        C = torch.zeros(m, l, dtype=torch.float64, device=DEV)
        for i in range(N + e):
            w = (mask[:, :, i] / mask.sum(2)).repeat_interleave(b, 0)[:m]
            w = w.repeat_interleave(b, 1)[:, :l]
            Y = _sketch64(A, seed, i, b)
            C += w * (Y @ (Y if Bt is A else _sketch64(Bt, seed, i, b)).t())
        return C
    A, B = _pair(case, g)
    keep = _keep(case, seed)[0]
    C = torch.zeros(m, l, dtype=torch.float64, device=DEV)
    At, Bt = [], []
    for i in range(N + e):
        if kind == "matmul" and not keep[i]:
            continue
        Ya, Yb = _sketch64(A, seed, i, b), _sketch64(B.t(), seed, i, b)
        if keep[i]:
            C += Ya @ Yb.t()
        if kind == "staged":
            pad = -b % 32
            At.append(torch.nn.functional.pad(Ya, (0, pad)))
            Bt.append(torch.nn.functional.pad(Yb, (0, pad)))
    C /= int(keep.sum())
    return C if kind == "matmul" else (torch.cat(At, 1), torch.cat(Bt, 1), C)
