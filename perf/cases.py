"""The work that a program has this library do, as timed cases.

Every case is one call of a public entry point on operands that are already on
the GPU: a single FT-GEMM (``ftgemm_run``, or ``ftgemm_matmul`` on row-major
tensors) in FP32, BF16 or FP8, one in FP64 or double complex
(``ftgemm_run_f64``, ``ftgemm_run_z64``), or a batch of problems of mixed sizes
and types (``ftgemm_batched``).  The fields of a case:

``entry``      run | matmul | f64 | z64 | batched
``dtype``      f32 | bf16 | fp8 (run, matmul); mix of a batch: f32+bf16 | f32+bf16+fp8
``m, n, k``    sizes; for a batch ``count``, ``lo, hi`` (range of every dimension)
               and ``shapes`` (the seed its sizes are drawn from)
``level``      0 plain, 1 detect only, 2 online detect and correct
``recompute``  FTGEMM_FT_RECOMPUTE on top of the level
``beta``       0 (C is written) or 1 (C is accumulated into, as the benchmark does)
``report``     the call fills a report (and so waits), as a program does that
               looks at every call's outcome; without it calls are queued

Matrices are packed: a leading dimension is the number of rows, so an odd size
also means operands whose columns are not aligned.
"""
import math

import numpy as np
import torch

from paper_2305_01024_amd import ftgemm as F

DTYPES = {"f32": F.F32, "bf16": F.BF16, "fp8": F.F8E4M3}
ELEMENT_BYTES = {"f32": 4, "bf16": 2, "fp8": 1}
E4M3_MAX = 448.0


def _single(name, entry, dtype, m, n, k, level=2, recompute=False, beta=0.0, report=False):
    c = {"entry": entry, "dtype": dtype, "m": m, "n": n, "k": k, "level": level, "recompute": recompute,
         "beta": beta, "report": report}
    return dict(c, name=name) if name else c


def listed():
    return [
        # a small product whose outcome is looked at after every call: latency
        _single("f32_256", "run", "f32", 256, 256, 256, report=True),
        # square FP32 products of the benchmark, accumulated into C
        _single("f32_2048", "run", "f32", 2048, 2048, 2048, beta=1.0),
        _single("f32_8192", "run", "f32", 8192, 8192, 8192, beta=1.0),
        # the benchmark's irregular shapes: tall and skinny, short inner
        # dimension, and sizes that divide by nothing
        _single("f32_tall", "run", "f32", 65536, 256, 4096),
        _single("f32_small_k", "run", "f32", 16384, 16384, 64),
        _single("f32_odd", "run", "f32", 3001, 1999, 4097),
        # a BF16 layer of a PyTorch program: row-major tensors, flagged tiles recomputed
        _single("bf16_2048", "matmul", "bf16", 2048, 2048, 2048, recompute=True),
        # the benchmark's large low-precision products
        _single("bf16_8192", "run", "bf16", 8192, 8192, 8192),
        _single("fp8_8192", "run", "fp8", 8192, 8192, 8192),
        # BF16 with sizes that divide by nothing, detection only
        _single("bf16_odd", "run", "bf16", 3001, 1999, 4097, level=1),
        # double precision
        _single("f64_4096", "f64", "f64", 4096, 4096, 4096, beta=1.0),
        # the benchmark's batch: 1024 problems, dimensions log-uniform in [32, 2048]
        {"name": "batched_1024", "entry": "batched", "dtype": "f32+bf16", "count": 1024, "lo": 32, "hi": 2048,
         "shapes": 5, "level": 2},
    ]


def _size(rng, lo, hi):
    """Log-uniform; half of the sizes as they come, half on a multiple of 64
    (of 16 below 128), as layer widths are."""
    x = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    if rng.random() < 0.5:
        step = 64 if x >= 128 else 16
        return max(lo, int(round(x / step)) * step)
    return max(lo, int(round(x)))


def draw(rng):
    level = rng.choice([2, 2, 2, 2, 1, 0])
    u = rng.random()
    if u < 0.15:
        return {"entry": "batched", "dtype": rng.choice(["f32+bf16", "f32+bf16", "f32+bf16+fp8"]),
                "count": int(round(math.exp(rng.uniform(math.log(16), math.log(1024))))), "lo": 32, "hi": 2048,
                "shapes": rng.randrange(1000), "level": level}
    beta = rng.choice([0.0, 1.0])
    report = rng.random() < 0.25
    if u < 0.27:
        entry, dtype, hi, recompute = rng.choice(["f64", "f64", "z64"]), "f64", 4096, False
        if entry == "z64":
            dtype, hi = "c64", 2048
    else:
        entry = rng.choice(["run", "run", "matmul"])
        dtype = rng.choice(["f32", "f32", "bf16", "bf16", "fp8"])
        recompute = level > 0 and rng.random() < 0.25
        hi = 8192
    m, n, k = (_size(rng, 64, hi) for _ in range(3))
    if rng.random() < 0.35:   # a square product
        n = k = m
    return _single(None, entry, dtype, m, n, k, level, recompute, beta, report)


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
class _Handle:
    """A library handle that goes with the state that holds it."""

    def __init__(self, dtype):
        self.h = F.ftgemm_create(dtype, torch.cuda.current_device())

    def __del__(self):
        F.ftgemm_destroy(self.h)


def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _normal(shape, g, dtype=torch.float32):
    return torch.randn(shape, generator=g, device="cuda", dtype=dtype)


def _heavy_tailed(shape, g):
    """N(0, 1) with 1% of the entries 100 times as large, as activations are."""
    x = _normal(shape, g)
    x[torch.rand(shape, generator=g, device="cuda") < 0.01] *= 100.0
    return x


def _operand(shape, dtype, g):
    """An operand of the case's type and its per-tensor scale (a power of two)."""
    if dtype == "f32":
        return _normal(shape, g), 1.0
    x = _heavy_tailed(shape, g)
    if dtype == "bf16":
        return x.to(torch.bfloat16), 1.0
    s = 2.0 ** math.ceil(math.log2(float(x.abs().max()) / E4M3_MAX))
    return (x / s).to(torch.float8_e4m3fn), s


def _batch_problems(case):
    """Sizes and types of a batch's problems (the same for every seed),
    dimensions log-uniform."""
    r = np.random.default_rng(case["shapes"])
    dims = np.rint(np.exp(r.uniform(np.log(case["lo"]), np.log(case["hi"]), size=(case["count"], 3)))).astype(int)
    kinds = case["dtype"].split("+")
    return [(int(m), int(n), int(k), kinds[int(t)]) for (m, n, k), t in zip(dims, r.integers(0, len(kinds), len(dims)))]


class _Pool:
    """One buffer that holds a list of matrices, each on a 256-byte boundary."""

    def __init__(self, sizes, bytes_each):
        step = 256 // bytes_each
        self.at, total = [], 0
        for s in sizes:
            self.at.append(total)
            total += -(-s // step) * step
        self.total, self.sizes = max(1, total), sizes

    def view(self, buf, q):
        return buf[self.at[q]: self.at[q] + self.sizes[q]]


def _batch_operands(case, seed):
    """Per type: the pooled A and B operands and their scales; C's pool."""
    probs, g = _batch_problems(case), _generator(seed)
    ops = {}
    for kind in case["dtype"].split("+"):
        mine = [p for p in probs if p[3] == kind]
        pa = _Pool([m * k for m, n, k, _ in mine], ELEMENT_BYTES[kind])
        pb = _Pool([k * n for m, n, k, _ in mine], ELEMENT_BYTES[kind])
        (a, sa), (b, sb) = _operand((pa.total,), kind, g), _operand((pb.total,), kind, g)
        ops[kind] = (pa, a, sa, pb, b, sb)
    return probs, ops, _Pool([m * n for m, n, _, _ in probs], 4)


def _single_operands(case, seed):
    """Operands as stored: dA holds the column-major m x k matrix as (k, m), dB
    the k x n one as (n, k), dC as (n, m).  matmul takes row-major tensors,
    (m, k), (k, n) and (m, n)."""
    g, m, n, k = _generator(seed), case["m"], case["n"], case["k"]
    rows = case["entry"] == "matmul"
    sa, sb, sc = ((m, k), (k, n), (m, n)) if rows else ((k, m), (n, k), (n, m))
    if case["dtype"] in ("f64", "c64"):
        t = torch.float64 if case["dtype"] == "f64" else torch.complex128
        a, b, scale = _normal(sa, g, t), _normal(sb, g, t), 1.0
    else:
        t = torch.float32
        (a, fa), (b, fb) = _operand(sa, case["dtype"], g), _operand(sb, case["dtype"], g)
        scale = (fa, fb)
    c = _normal(sc, g, t) if case["beta"] else torch.zeros(sc, device="cuda", dtype=t)
    return a, b, c, scale


def prepare(case, seed):
    if case["entry"] == "batched":
        probs, ops, pc = _batch_operands(case, seed)
        c = torch.zeros(pc.total, device="cuda")
        at = {kind: 0 for kind in ops}
        desc = F.make_problems(len(probs))
        for q, (m, n, k, kind) in enumerate(probs):
            pa, a, sa, pb, b, sb = ops[kind]
            x, size = at[kind], ELEMENT_BYTES[kind]
            at[kind] += 1
            desc[q] = (DTYPES[kind], 0, m, n, k, m, k, m, 1.0, 0.0, sa, sb, a.data_ptr() + pa.at[x] * size,
                       b.data_ptr() + pb.at[x] * size, c.data_ptr() + pc.at[q] * 4)
        return {"case": case, "handle": _Handle(F.F32), "problems": desc, "keep": ops, "C": c}
    a, b, c, scale = _single_operands(case, seed)
    kind = {"f64": F.F64, "c64": F.C64}.get(case["dtype"])
    handle = _Handle(DTYPES[case["dtype"]] if kind is None else kind)
    if case["dtype"] == "fp8":
        F.ftgemm_set_scales(handle.h, *scale)
    rep = F.ReportBuffer(1024) if case["report"] else None
    return {"case": case, "handle": handle, "A": a, "B": b, "C": c, "report": rep}


def run(state):
    case, h, c = state["case"], state["handle"].h, state["C"]
    if case["entry"] == "batched":
        F.ftgemm_batched(h, state["problems"], case["level"], 0.0, torch.cuda.current_stream().cuda_stream)
        return c
    a, b, rep = state["A"], state["B"], state["report"]
    m, n, k, beta = case["m"], case["n"], case["k"], case["beta"]
    level = case["level"] | (F.FT_RECOMPUTE if case["recompute"] else 0)
    if case["entry"] == "matmul":
        F.ftgemm_matmul(h, a, b, c, 1.0, beta, level, 0.0, rep)
    else:
        call = {"run": F.ftgemm_run, "f64": F.ftgemm_run_f64, "z64": F.ftgemm_run_z64}[case["entry"]]
        call(h, m, n, k, 1.0, a.data_ptr(), m, b.data_ptr(), k, beta, c.data_ptr(), m, level, 0.0,
             torch.cuda.current_stream().cuda_stream, rep)
    if rep is None:
        return c
    r = rep.report
    return {"C": c, "outcome": [int(r.detected), int(r.corrected), int(r.uncorrectable), int(r.nonfinite_input)]}


def work(case):
    if case["entry"] == "batched":
        probs = _batch_problems(case)
        return {"bytes": sum(ELEMENT_BYTES[t] * (m * k + k * n) + 4 * m * n for m, n, k, t in probs),
                "flops": sum(2 * m * n * k for m, n, k, _ in probs)}
    m, n, k = case["m"], case["n"], case["k"]
    e = {"f64": 8, "c64": 16}.get(case["dtype"]) or ELEMENT_BYTES[case["dtype"]]
    out = {"f64": 8, "c64": 16}.get(case["dtype"], 4)
    reads = 2 if case["beta"] else 1
    return {"bytes": e * (m * k + k * n) + out * reads * m * n,
            "flops": (8 if case["dtype"] == "c64" else 2) * m * n * k}


def exact(case, seed):
    """The products in 64 bits with torch, from the stored operands."""
    if case["entry"] == "batched":
        probs, ops, pc = _batch_operands(case, seed)
        out, at = torch.zeros(pc.total, device="cuda", dtype=torch.float64), {kind: 0 for kind in ops}
        for q, (m, n, k, kind) in enumerate(probs):
            pa, a, sa, pb, b, sb = ops[kind]
            x = at[kind]
            at[kind] += 1
            ca = pa.view(a, x).double().view(k, m)
            cb = pb.view(b, x).double().view(n, k)
            pc.view(out, q).view(n, m).copy_((cb @ ca) * (sa * sb))
        return out
    a, b, c, scale = _single_operands(case, seed)
    wide = torch.complex128 if case["dtype"] == "c64" else torch.float64
    factor = scale[0] * scale[1] if isinstance(scale, tuple) else 1.0
    a, b, c = a.to(wide), b.to(wide), c.to(wide)
    p = a @ b if case["entry"] == "matmul" else b @ a
    p = p * factor + case["beta"] * c
    return {"C": p, "outcome": None} if case["report"] else p
