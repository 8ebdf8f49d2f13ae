"""The work that programs have this library do, as cases a timer can run.

Each case is one call (or one data region) through the public entry points,
over the sizes, element types, value distributions and options that the
repository's own configurations use: the loop-nest matmul of Listing 1a
(section 1.3) from LEN = 64 to 8192 in float32 and int32, rectangular nests,
reductions from 2^12 to 2^28 elements, a matmul and a reduction in one
region, batches, and the data directive around host arrays.

listed() gives the cases, draw() further ones of the same ranges, prepare()
what a program holds before the call (device arrays, caller workspaces, a
batch plan), run() the call, work() the bytes and operations it cannot do
without, and exact() the results in float64.

The tile autotuner is not run for single calls: it is an option, and its
table is one per process, so that it would carry over from case to case.
"""
import math

import numpy as np
import torch

import paper_1412_1127_amd as ax

_F32, _I32 = "float32", "int32"
_DTYPES = {
    "float32": (ax.ACC_FLOAT32, torch.float32, 4),
    "int32": (ax.ACC_INT32, torch.int32, 4),
    "float64": (ax.ACC_FLOAT64, torch.float64, 8),
    "int64": (ax.ACC_INT64, torch.int64, 8),
}
_PREC = {"auto": ax.ACC_PREC_AUTO, "full6": ax.ACC_PREC_FULL6}
# reduction variables: (operator, square)
_VARS = {
    "sum": [(ax.ACC_RED_SUM, 0)],
    "sum_sumsq": [(ax.ACC_RED_SUM, 0), (ax.ACC_RED_SUM, 1)],  # the SRAD loop's pair
    "max_min": [(ax.ACC_RED_MAX, 0), (ax.ACC_RED_MIN, 0)],
}
_ready = False


def listed():
    return [
        # The smallest configuration: one LEN = 256 nest, where launches and
        # latency are all there is.
        {"name": "matmul_f32_256", "kind": "matmul", "dtype": _F32, "m": 256, "n": 256, "k": 256, "pad": 0,
         "prec": "auto", "values": "uniform"},
        # An ordinary size that no tile divides (the paper's own benchmark is
        # 1024 x 1024).
        {"name": "matmul_f32_1000", "kind": "matmul", "dtype": _F32, "m": 1000, "n": 1000, "k": 1000, "pad": 0,
         "prec": "auto", "values": "uniform"},
        # The top of the serving range, at the precision that needs no probe.
        {"name": "matmul_f32_full6_2048", "kind": "matmul", "dtype": _F32, "m": 2048, "n": 2048, "k": 2048, "pad": 0,
         "prec": "full6", "values": "uniform"},
        # The precision configuration, the largest case: normal values times
        # a power of two per row, where the probe marks tiles for correction.
        {"name": "matmul_f32_8192_rowscaled", "kind": "matmul", "dtype": _F32, "m": 8192, "n": 8192, "k": 8192,
         "pad": 0, "prec": "auto", "values": "rowscaled"},
        # One GPU's rows of a LEN = 4096 nest shared over eight: few output
        # tiles, views into larger arrays.
        {"name": "gemm_f32_512x4096x4096", "kind": "matmul", "dtype": _F32, "m": 512, "n": 4096, "k": 4096, "pad": 64,
         "prec": "auto", "values": "uniform"},
        # The int32 nest of the scale configuration: values that one int8
        # digit holds.
        {"name": "matmul_i32_4096", "kind": "matmul", "dtype": _I32, "m": 4096, "n": 4096, "k": 4096, "pad": 0,
         "prec": "auto", "values": "pm16"},
        # The same nest on arbitrary integers (four digits), at a ragged size.
        {"name": "matmul_i32_full_1531", "kind": "matmul", "dtype": _I32, "m": 1531, "n": 1531, "k": 1531, "pad": 0,
         "prec": "auto", "values": "full"},
        # The benchmark's default step: float32 LEN = 4096 and the sum of
        # 2^28 floats as one region.
        {"name": "matmul_reduce_4096", "kind": "matmul_reduce", "len": 4096, "n": 1 << 28},
        # A short reduction: the low end of the serving and batch range.
        {"name": "sum_f32_100003", "kind": "reduce", "dtype": _F32, "n": 100003, "vars": "sum"},
        # The SRAD loop's sum and sum of squares over a large image.
        {"name": "sumsq_f32_16m", "kind": "reduce", "dtype": _F32, "n": 1 << 24, "vars": "sum_sumsq"},
        # The batching configuration: 512 matmuls and 256 reductions in one
        # graph launch.
        {"name": "batch_512_256", "kind": "batch", "mats": 512, "reds": 256, "max_len": 1024, "step": 64},
        # The paper's program: a data region around a 1024 x 1024 nest on
        # host arrays, with a reduction over a fourth.
        {"name": "region_1024", "kind": "region", "dtype": _F32, "len": 1024},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["matmul", "matmul", "gemm", "matmul_i32", "matmul_i32", "reduce", "reduce", "matmul_reduce",
                       "batch", "region"])
    if kind == "matmul":
        n = _log_int(rng, 64, 4096)
        return {"kind": "matmul", "dtype": _F32, "m": n, "n": n, "k": n, "pad": 0,
                "prec": rng.choice(["auto", "auto", "full6"]), "values": rng.choice(["uniform", "uniform", "rowscaled"])}
    if kind == "gemm":
        return {"kind": "matmul", "dtype": rng.choice([_F32, _F32, _I32]), "m": _log_int(rng, 32, 4096),
                "n": _log_int(rng, 32, 4096), "k": _log_int(rng, 32, 4096), "pad": rng.choice([0, 3, 64]),
                "prec": "auto", "values": "uniform"}
    if kind == "matmul_i32":
        n = _log_int(rng, 64, 4096)
        return {"kind": "matmul", "dtype": _I32, "m": n, "n": n, "k": n, "pad": 0, "prec": "auto",
                "values": rng.choice(["pm16", "pm16", "pm20000", "full"])}
    if kind == "reduce":
        return {"kind": "reduce", "dtype": rng.choice([_F32, _F32, _I32, "float64", "int64"]),
                "n": _log_int(rng, 1 << 12, 1 << 27), "vars": rng.choice(["sum", "sum", "sum_sumsq", "max_min"])}
    if kind == "matmul_reduce":
        return {"kind": "matmul_reduce", "len": _log_int(rng, 256, 4096), "n": _log_int(rng, 1 << 16, 1 << 28)}
    if kind == "batch":
        return {"kind": "batch", "mats": _log_int(rng, 16, 512), "reds": _log_int(rng, 8, 256),
                "max_len": rng.choice([256, 512, 1024]), "step": rng.choice([1, 64])}
    return {"kind": "region", "dtype": rng.choice([_F32, _F32, _I32]), "len": _log_int(rng, 128, 2048)}


# ---- inputs ----------------------------------------------------------------

def _gen(seed, stream):
    g = torch.Generator(device="cuda")
    g.manual_seed((int(seed) * 1000003 + stream) & 0x7fffffffffffffff)
    return g


def _uniform_pm1(shape, seed, stream):
    return torch.rand(shape, generator=_gen(seed, stream), device="cuda") * 2 - 1


def _matrix(dtype, values, rows, cols, seed, stream):
    if dtype == _F32:
        if values == "rowscaled":  # N(0, 1) * 2^U(-8, 8) per row, rounded once
            g = _gen(seed, stream)
            z = torch.randn((rows, cols), generator=g, device="cuda", dtype=torch.float64)
            u = torch.rand((rows, 1), generator=g, device="cuda", dtype=torch.float64) * 16 - 8
            return z.mul_(torch.exp2(u)).float()
        return _uniform_pm1((rows, cols), seed, stream)
    lo, hi = {"pm20000": (-20000, 20000), "full": (-(1 << 31), (1 << 31) - 1)}.get(values, (-16, 16))
    return torch.randint(lo, hi + 1, (rows, cols), generator=_gen(seed, stream), device="cuda",
                         dtype=torch.int64).to(torch.int32)


def _strided(x, pad):
    """x as a view into an array whose rows are `pad` elements longer."""
    if not pad:
        return x
    big = torch.zeros((x.shape[0], x.shape[1] + pad), dtype=x.dtype, device=x.device)
    big[:, :x.shape[1]] = x
    return big[:, :x.shape[1]]


def _vector(dtype, n, seed, stream):
    if dtype in ("float32", "float64"):
        return torch.rand(n, generator=_gen(seed, stream), device="cuda", dtype=_DTYPES[dtype][1])
    return torch.randint(-(1 << 31), 1 << 31, (n,), generator=_gen(seed, stream), device="cuda",
                         dtype=torch.int64).to(_DTYPES[dtype][1])


def _matmul_inputs(case, seed):
    a = _matrix(case["dtype"], case["values"], case["m"], case["k"], seed, 1)
    b = _matrix(case["dtype"], case["values"], case["k"], case["n"], seed, 2)
    return a, b


def _batch_sizes(case):
    """LEN uniform over the multiples of `step`, n log-uniform, fixed per case: a batch is planned once."""
    g = np.random.Generator(np.random.PCG64([case["mats"], case["reds"], case["max_len"], case["step"]]))
    lo = max(case["step"], 64)
    lens = g.integers(lo // case["step"], case["max_len"] // case["step"] + 1, case["mats"]) * case["step"]
    ns = np.exp(g.uniform(math.log(1 << 16), math.log(1 << 24), case["reds"])).astype(np.int64)
    return [int(v) for v in lens], [int(v) for v in ns]


def _offsets(counts):
    """Element offsets of consecutive arrays, each starting on a 256-byte boundary, and their total."""
    off, out = 0, []
    for c in counts:
        out.append(off)
        off += (c + 63) // 64 * 64
    return out, off


def _batch_inputs(case, seed):
    lens, ns = _batch_sizes(case)
    offs, total = _offsets([v * v for v in lens])
    xoffs, xtotal = _offsets(ns)
    a = _uniform_pm1((total,), seed, 1)
    b = _uniform_pm1((total,), seed, 2)
    x = torch.rand(xtotal, generator=_gen(seed, 3), device="cuda")
    return lens, ns, offs, xoffs, a, b, x


def _region_inputs(case, seed):
    n = case["len"]
    a = _matrix(case["dtype"], "uniform", n, n, seed, 1).cpu().numpy()
    b = _matrix(case["dtype"], "uniform", n, n, seed, 2).cpu().numpy()
    return a, b, _vector(case["dtype"], n * n, seed, 3).cpu().numpy()


# ---- the cases --------------------------------------------------------------

class _Batch:
    """A planned batch and the arrays it is bound to."""

    def __init__(self, case, seed):
        lens, ns, offs, xoffs, self.a, self.b, self.x = _batch_inputs(case, seed)
        self.c = torch.zeros_like(self.a)
        self.results = torch.zeros(len(ns), device="cuda")
        items = [ax.batch_matmul(self.a[o:], self.b[o:], self.c[o:], n) for n, o in zip(lens, offs)]
        items += [ax.batch_reduce(self.x[o:], n, self.results[k:]) for k, (n, o) in enumerate(zip(ns, xoffs))]
        self.handle = ax.accx_batch_create(items, ax.ACC_BATCH_AUTOTUNE | ax.ACC_BATCH_PREC_AUTO)

    def __del__(self):
        if getattr(self, "handle", None):
            ax.accx_batch_destroy(self.handle)


def prepare(case, seed):
    global _ready
    if not _ready:
        ax.acc_init(torch.cuda.current_device(), 0)
        _ready = True
    kind = case["kind"]
    st = {"case": case}
    if kind == "matmul":
        t, tt, _ = _DTYPES[case["dtype"]]
        m, n, k, pad = case["m"], case["n"], case["k"], case["pad"]
        a, b = _matmul_inputs(case, seed)
        st["a"], st["b"] = _strided(a, pad), _strided(b, pad)
        st["out"] = torch.empty((m, n), dtype=tt, device="cuda")
        st["flags"] = _PREC[case["prec"]]
        st["bytes"] = ax.accx_gemm_workspace_size(t, m, n, k, st["flags"])
        st["work"] = torch.empty(max(1, st["bytes"]), dtype=torch.uint8, device="cuda")
    elif kind == "matmul_reduce":
        n = case["len"]
        st["a"], st["b"] = _uniform_pm1((n, n), seed, 1), _uniform_pm1((n, n), seed, 2)
        st["x"] = _vector(_F32, case["n"], seed, 3)
        st["out"] = torch.empty((n, n), device="cuda")
        st["sum"] = torch.empty(1, device="cuda")
        st["bytes"] = ax.accx_matmul_reduce_workspace_size(n, 0, case["n"])
        st["work"] = torch.empty(st["bytes"], dtype=torch.uint8, device="cuda")
    elif kind == "reduce":
        t, tt, _ = _DTYPES[case["dtype"]]
        st["x"] = _vector(case["dtype"], case["n"], seed, 3)
        st["vars"] = _VARS[case["vars"]]
        st["init"] = [0] * len(st["vars"])
        st["out"] = torch.empty(len(st["vars"]), dtype=tt, device="cuda")
        st["bytes"] = ax.accx_reduce_vars_workspace_size(t, case["n"], st["vars"])
        st["work"] = torch.empty(st["bytes"], dtype=torch.uint8, device="cuda")
    elif kind == "batch":
        st["batch"] = _Batch(case, seed)
    else:
        st["a"], st["b"], st["x"] = _region_inputs(case, seed)
        st["out"] = np.zeros_like(st["a"])
        st["sum"] = np.zeros(1, dtype=st["a"].dtype)
    return st


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "matmul":
        t = _DTYPES[case["dtype"]][0]
        a, b, c = st["a"], st["b"], st["out"]
        m, n, k = case["m"], case["n"], case["k"]
        if m == n == k and not case["pad"]:
            ax.accx_matmul_dev(t, a, b, c, n, st["flags"], st["work"], st["bytes"])
        else:
            ax.accx_gemm_dev(t, m, n, k, a, a.stride(0), b, b.stride(0), c, n, st["flags"], st["work"], st["bytes"])
        return c
    if kind == "matmul_reduce":
        ax.accx_matmul_reduce_dev(st["a"], st["b"], st["out"], case["len"], 0, st["x"], case["n"], 0.0, st["sum"],
                                  st["work"], st["bytes"])
        return [st["out"], st["sum"]]
    if kind == "reduce":
        ax.accx_reduce_dev(_DTYPES[case["dtype"]][0], st["x"], case["n"], st["vars"], st["init"], st["out"], 0,
                           st["work"], st["bytes"])
        return st["out"]
    if kind == "batch":
        ax.accx_batch_launch(st["batch"].handle)
        return [st["batch"].c, st["batch"].results]
    t = _DTYPES[case["dtype"]][0]
    a, b, c, x, s, n = st["a"], st["b"], st["out"], st["x"], st["sum"], case["len"]
    s[0] = 0
    region = ax.acc_data_begin([ax.clause(ax.ACC_COPYIN, t, a), ax.clause(ax.ACC_COPYIN, t, b),
                                ax.clause(ax.ACC_COPYOUT, t, c), ax.clause(ax.ACC_COPYIN, t, x)])
    ax.acc_loopnest_matmul(region, t, a, b, c, n)
    ax.acc_reduce_sum(region, t, x, n * n, s)
    ax.acc_data_end(region)
    return [c, s]


def work(case):
    """Each input read once, each result written once; 2 operations per step of the nest, as the nest states them
    (float32 on bf16 matrix cores runs at least three products for each)."""
    kind = case["kind"]
    if kind == "matmul":
        m, n, k = case["m"], case["n"], case["k"]
        return {"bytes": 4 * (m * k + k * n + m * n), "flops": 2 * m * n * k}
    if kind == "matmul_reduce":
        n = case["len"]
        return {"bytes": 12 * n * n + 4 * case["n"], "flops": 2 * n ** 3 + case["n"]}
    if kind == "reduce":
        return {"bytes": case["n"] * _DTYPES[case["dtype"]][2], "flops": case["n"] * len(_VARS[case["vars"]])}
    if kind == "batch":
        lens, ns = _batch_sizes(case)
        return {"bytes": sum(12 * v * v for v in lens) + 4 * sum(ns), "flops": sum(2 * v ** 3 for v in lens) + sum(ns)}
    n = case["len"]
    return {"bytes": 16 * n * n, "flops": 2 * n ** 3 + n * n}


def exact(case, seed):
    """run()'s results in float64; integer results have none (they are exact as they are)."""
    kind = case["kind"]
    if case.get("dtype") in ("int32", "int64"):
        return None
    if kind == "matmul":
        a, b = _matmul_inputs(case, seed)
        return a.double() @ b.double()
    if kind == "matmul_reduce":
        n = case["len"]
        a, b = _uniform_pm1((n, n), seed, 1), _uniform_pm1((n, n), seed, 2)
        return [a.double() @ b.double(), _vector(_F32, case["n"], seed, 3).sum(dtype=torch.float64).reshape(1)]
    if kind == "reduce":
        x = _vector(case["dtype"], case["n"], seed, 3).double()
        if case["vars"] == "max_min":
            return torch.stack([x.max(), x.min()])
        # a squared term is rounded in the element type before it is folded
        return torch.stack([x.sum()] + ([(x.to(_DTYPES[case["dtype"]][1]) ** 2).double().sum()]
                                        if case["vars"] == "sum_sumsq" else []))
    if kind == "batch":
        lens, ns, offs, xoffs, a, b, x = _batch_inputs(case, seed)
        c = torch.zeros_like(a, dtype=torch.float64)
        for n, o in zip(lens, offs):
            c[o:o + n * n] = (a[o:o + n * n].view(n, n).double() @ b[o:o + n * n].view(n, n).double()).reshape(-1)
        return [c, torch.stack([x[o:o + n].sum(dtype=torch.float64) for n, o in zip(ns, xoffs)])]
    a, b, x = (torch.from_numpy(v).cuda() for v in _region_inputs(case, seed))
    return [a.double() @ b.double(), x.sum(dtype=torch.float64).reshape(1)]
