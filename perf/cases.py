"""The work a user of this framework has it do, as measurable cases.

Every case goes through the package's public entry points on tensors the caller
owns: single products C = alpha*A*B + beta*C (``gemm``, FP64, FP32 and the
emulated FP64 types), lists of uneven products (``gemm_batched`` for a list used
once, ``BatchedPlan`` for one that is executed again and again) and the training
of the tile-choice network (``MLP``).

Sizes are those of the repository's benchmark, tests and tuner: squares from 256
to 8192, shapes with m, n, k log-uniform in [64, 16384], outputs of few tiles
with a long k, 2048 problems with m, n, k log-uniform in [16, 1024], and the
network 6 -> 64 -> 64 -> 247 on 13600 rows.  Dense values are uniform in [-1, 1);
the emulated types get u * 2^e with e in [-20, 20], the range they are meant for.
"""
import math
import random

import numpy as np
import torch

import paper_1706_10086_amd as mg

DTYPES = {"f64": mg.F64, "f32": mg.F32, "split_bf16": mg.SPLIT_BF16, "split_fp8": mg.SPLIT_FP8,
          "split_int8": mg.SPLIT_INT8, "crt_int8": mg.CRT_INT8}
# low-precision products each emulated type forms per product of A and B (the
# kept slice pairs of 6, 11 and 8 slices; one per modulus)
PRODUCTS = {"f64": 1, "f32": 1, "split_bf16": 21, "split_fp8": 66, "split_int8": 36,
            "crt_int8": 16}
LARGEST_FLOPS = 2.0 * 8192 ** 3
MLP_DIMS = (6, 64, 247)


def _gemm(name, dtype, m, n, k, alpha=1.0, beta=0.5, pad=0):
    return {"name": name, "kind": "gemm", "dtype": dtype, "m": m, "n": n, "k": k,
            "alpha": alpha, "beta": beta, "pad": pad}


def _batch(name, kind, dtype, count, lo, hi, shapes):
    return {"name": name, "kind": kind, "dtype": dtype, "count": count, "lo": lo, "hi": hi,
            "shapes": shapes, "alpha": 1.0, "beta": 0.0}


def listed():
    return [
        # one small product per call, the parity size: latency and launch cost
        _gemm("f64_256", "f64", 256, 256, 256, 1.5, 0.5),
        # the headline: a large square product that fills the GPU for many rounds
        _gemm("f64_8192", "f64", 8192, 8192, 8192),
        # an ordinary product of odd sizes (rows that are no whole 16-byte loads),
        # as most of the tuner's shapes are
        _gemm("f64_ragged", "f64", 1999, 1501, 2777),
        # few outputs and a long sum (a projection onto a small basis)
        _gemm("f64_thin", "f64", 300, 129, 10007),
        # the smallest square of the benchmark's sweep, in FP32
        _gemm("f32_1024", "f32", 1024, 1024, 1024),
        # FP32 on a block of a wider matrix (leading dimensions beyond the row)
        _gemm("f32_ragged", "f32", 3001, 777, 1211, pad=6),
        # FP64-accurate products from int8 residues: the fastest emulation
        _gemm("crt_int8_4096", "crt_int8", 4096, 4096, 4096, beta=0.0),
        # the same from int8 slices, odd sizes
        _gemm("split_int8_ragged", "split_int8", 1500, 2301, 3107, beta=0.0),
        # the same from bfloat16 slices
        _gemm("split_bf16_2048", "split_bf16", 2048, 2048, 2048, beta=0.0),
        # thousands of uneven products with a plan kept between executions
        _batch("plan_f64_2048", "plan", "f64", 2048, 16, 1024, 4),
        # a list of uneven products used once, no plan
        _batch("list_f32_100", "list", "f32", 100, 16, 1024, 7),
        # training the tile-choice network at its own size: 20 full-batch steps
        {"name": "mlp_train", "kind": "mlp", "rows": 13600, "hidden": 64, "out": 247, "steps": 20},
    ]


def _log_int(rng, lo, hi):
    return min(hi, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))


def draw(rng):
    kind = rng.choice(["square", "ragged", "ragged", "thin", "emulated", "plan", "list", "mlp"])
    if kind == "plan":
        c = _batch("", kind, rng.choice(["f64", "f32"]), _log_int(rng, 100, 2048), 16,
                   rng.choice([256, 512, 1024]), rng.randrange(1 << 20))
    elif kind == "list":
        c = _batch("", kind, rng.choice(["f64", "f32"]), _log_int(rng, 10, 150), 16,
                   rng.choice([256, 512, 1024]), rng.randrange(1 << 20))
    elif kind == "mlp":
        c = {"kind": "mlp", "rows": _log_int(rng, 500, 13600), "hidden": rng.choice([32, 64, 100]),
             "out": rng.randrange(20, 248), "steps": rng.randrange(1, 21)}
    elif kind == "emulated":
        dtype = rng.choice(["split_bf16", "split_fp8", "split_int8", "crt_int8"])
        m, n, k = (_log_int(rng, 128, 4096) for _ in range(3))
        c = _gemm("", dtype, m, n, k, 1.0, rng.choice([0.0, 0.5]), rng.choice([0, 0, 3]))
    else:
        dtype = rng.choice(["f64", "f32"])
        alpha, beta = rng.choice([(1.0, 0.0), (1.0, 0.5), (1.5, 0.5)])
        if kind == "square":
            m = n = k = 64 * _log_int(rng, 2, 126)
        elif kind == "thin":
            m, n, k = _log_int(rng, 16, 512), _log_int(rng, 16, 512), _log_int(rng, 2048, 16384)
        else:
            while True:
                m, n, k = (_log_int(rng, 64, 16384) for _ in range(3))
                if 2.0 * m * n * k <= LARGEST_FLOPS / 4:
                    break
        c = _gemm("", dtype, m, n, k, alpha, beta, rng.choice([0, 0, 0, 1, 8]))
    c.pop("name", None)
    return c


def _problems(case):
    """(m, n, k) of every product of a list or plan."""
    r = random.Random(case["shapes"])
    return [tuple(_log_int(r, case["lo"], case["hi"]) for _ in range(3))
            for _ in range(case["count"])]


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _uniform(shape, dtype, g, wide=False):
    x = torch.rand(shape, dtype=dtype, device="cuda", generator=g) * 2 - 1
    if wide:
        x = torch.ldexp(x, torch.randint(-20, 21, shape, device="cuda", generator=g))
    return x


def _matrix(rows, cols, pad, dtype, g, wide=False):
    """rows x cols with a leading dimension of cols + pad."""
    return _uniform((rows, cols + pad), dtype, g, wide)[:, :cols]


def _gemm_inputs(case, seed):
    g = _gen(seed)
    wide = case["dtype"] not in ("f64", "f32")
    t = torch.float32 if case["dtype"] == "f32" else torch.float64
    m, n, k, pad = case["m"], case["n"], case["k"], case["pad"]
    return (_matrix(m, k, pad, t, g, wide), _matrix(k, n, pad, t, g, wide),
            _matrix(m, n, pad, t, g))


def _arena(sizes, dtype, g=None):
    """Matrices of the given sizes in one buffer, each on a 256-byte boundary; the
    buffer uniform random, or zero without a generator."""
    step = 256 // torch.empty((), dtype=dtype).element_size()
    at, offs = 0, []
    for r, c in sizes:
        offs.append(at)
        at += -(-r * c // step) * step
    buf = torch.zeros(at, dtype=dtype, device="cuda") if g is None else _uniform((at,), dtype, g)
    return buf, [buf[o:o + r * c].view(r, c) for o, (r, c) in zip(offs, sizes)]


def _batch_inputs(case, seed):
    g = _gen(seed)
    t = torch.float32 if case["dtype"] == "f32" else torch.float64
    shapes = _problems(case)
    _, As = _arena([(m, k) for m, n, k in shapes], t, g)
    _, Bs = _arena([(k, n) for m, n, k in shapes], t, g)
    out, Cs = _arena([(m, n) for m, n, k in shapes], t)
    return As, Bs, Cs, out


def _mlp_inputs(case, seed):
    """Initial parameters (He uniform) and a training set: standardised features,
    targets in [0, 1], and a mask that leaves each row the outputs of one type."""
    g = _gen(seed)
    rows, hidden, out = case["rows"], case["hidden"], case["out"]
    r = np.random.RandomState(seed % (1 << 31))
    parts = []
    for fan, width in ((MLP_DIMS[0], hidden), (hidden, hidden), (hidden, out)):
        b = math.sqrt(6.0 / fan)
        parts += [r.uniform(-b, b, width * fan), np.zeros(width)]
    theta = np.concatenate(parts).astype(np.float32)
    X = torch.randn((rows, MLP_DIMS[0]), device="cuda", generator=g)
    T = torch.rand((rows, out), device="cuda", generator=g) ** 4
    first = torch.rand((rows, 1), device="cuda", generator=g) < 0.5
    M = (first == (torch.arange(out, device="cuda") < out // 2)[None, :]).float()
    return theta, X, T * M, M


def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case}
    if kind == "gemm":
        s["A"], s["B"], s["C"] = _gemm_inputs(case, seed)
    elif kind == "mlp":
        theta, X, T, M = _mlp_inputs(case, seed)
        s["net"] = mg.MLP(MLP_DIMS[0], case["hidden"], case["out"], theta)
        s["net"].set_data(X, T, M)
    else:
        s["As"], s["Bs"], s["Cs"], s["out"] = _batch_inputs(case, seed)
        if kind == "plan":
            s["plan"] = mg.BatchedPlan(s["As"], s["Bs"], s["Cs"], case["alpha"], case["beta"])
        else:
            mg.set_stream(torch.cuda.current_stream())
    return s


def run(s):
    case = s["case"]
    if case["kind"] == "gemm":
        return mg.gemm(s["A"], s["B"], s["C"], case["alpha"], case["beta"], DTYPES[case["dtype"]])
    if case["kind"] == "plan":
        s["plan"].execute()
        return s["out"]
    if case["kind"] == "list":
        mg.gemm_batched(s["As"], s["Bs"], s["Cs"], case["alpha"], case["beta"])
        return s["out"]
    loss = s["net"].train(case["steps"])
    return {"loss": loss, "params": s["net"].get_params()}


def work(case):
    if case["kind"] == "gemm":
        m, n, k = case["m"], case["n"], case["k"]
        es = 4 if case["dtype"] == "f32" else 8
        return {"bytes": es * (m * k + k * n + m * n * (2 if case["beta"] else 1)),
                "flops": 2.0 * m * n * k * PRODUCTS[case["dtype"]]}
    if case["kind"] == "mlp":
        i, h, o, b = MLP_DIMS[0], case["hidden"], case["out"], case["rows"]
        # forward, backward to the activations, gradients of the weights
        flops = 2.0 * b * (3 * (h * h + h * o) + 2 * i * h)
        return {"bytes": case["steps"] * 4 * b * (i + 2 * o), "flops": case["steps"] * flops}
    es = 4 if case["dtype"] == "f32" else 8
    shapes = _problems(case)
    return {"bytes": es * sum(m * k + k * n + m * n for m, n, k in shapes),
            "flops": 2.0 * sum(m * n * k for m, n, k in shapes)}


def _exact_mlp(case, seed):
    theta, X, T, M = _mlp_inputs(case, seed)
    i, h, o = MLP_DIMS[0], case["hidden"], case["out"]
    p = torch.from_numpy(theta).cuda().double()
    X, T, M = X.double(), T.double(), M.double()
    cuts = np.cumsum([h * i, h, h * h, h, o * h, o])[:-1].tolist()
    mom, var, loss = torch.zeros_like(p), torch.zeros_like(p), 0.0
    for t in range(1, case["steps"] + 1):
        W1, b1, W2, b2, W3, b3 = torch.tensor_split(p, cuts)
        W1, W2, W3 = W1.view(h, i), W2.view(h, h), W3.view(o, h)
        z1 = X @ W1.T + b1
        z2 = z1.clamp(min=0) @ W2.T + b2
        D = M * (z2.clamp(min=0) @ W3.T + b3 - T)
        loss = float((D * D).sum() / M.sum())
        dY = D * (2.0 / M.sum())
        dz2 = (dY @ W3) * (z2 > 0)
        dz1 = (dz2 @ W2) * (z1 > 0)
        g = torch.cat([(dz1.T @ X).reshape(-1), dz1.sum(0), (dz2.T @ z1.clamp(min=0)).reshape(-1),
                       dz2.sum(0), (dY.T @ z2.clamp(min=0)).reshape(-1), dY.sum(0)])
        mom = 0.9 * mom + 0.1 * g
        var = 0.999 * var + 0.001 * g * g
        p = p - 1e-3 * (mom / (1 - 0.9 ** t)) / ((var / (1 - 0.999 ** t)).sqrt() + 1e-8)
    return {"loss": loss, "params": p.cpu().numpy()}


def exact(case, seed):
    if case["kind"] == "gemm":
        A, B, C = (x.double() for x in _gemm_inputs(case, seed))
        return case["alpha"] * (A @ B) + case["beta"] * C
    if case["kind"] == "mlp":
        return _exact_mlp(case, seed)
    As, Bs, Cs, _ = _batch_inputs(case, seed)
    out, Xs = _arena([tuple(c.shape) for c in Cs],
                     torch.float32 if case["dtype"] == "f32" else torch.float64)
    out = out.double()
    for a, b, c in zip(As, Bs, Xs):
        out[c.storage_offset():c.storage_offset() + c.numel()] = (
            case["alpha"] * (a.double() @ b.double())).reshape(-1)
    return out
