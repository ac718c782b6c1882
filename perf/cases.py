"""The problems this library is timed on: Kron-Matmuls of the sizes its users run, through its public calls.

A case is one Kron-Matmul Y = X (F1 (x) ... (x) FN).  Its fields: `m` (rows of X), `factors` (the shapes, as
"8x8^6" or "52x50,65x20", in the order of the product), `dtype`, and `call`, the way a program makes it:

  prepared    arguments marshalled once into a Prepared call with its own workspace (iterative solvers)
  plain       kronmatmul(X, Fs): result and workspace come from the library and its binding
  buffers     kronmatmul with the caller's result and workspace tensors
  gradient    the backward direction, dX = dY (F1^T (x) ... (x) FN^T), from the factors of the forward product

Shapes are those of the repository's measured workloads, of the paper's Table 3, Table 4 and Figure 9 and of
the shape tables kept with the kernels."""
import math

import torch

import paper_2401_10187_amd as km


def listed():
    return [
        # one step of an iterative solver on a small grid: a single launch, all latency
        {"name": "solver_8x8x3", "m": 16, "factors": "8x8^3", "dtype": "float32", "call": "prepared"},
        # a real-world size of Table 4 (id 6): two different rectangular factors on a few rows, called as is
        {"name": "rect_52x50_65x20", "m": 10, "factors": "52x50,65x20", "dtype": "float32", "call": "plain"},
        # Table 4 id 18: many rows that fit on chip, small factors
        {"name": "rows_4x4x7", "m": 1024, "factors": "4x4^7", "dtype": "float32", "call": "buffers"},
        # the headline microbenchmark: rows of a megabyte, small factors
        {"name": "grid_8x8x6", "m": 1024, "factors": "8x8^6", "dtype": "float32", "call": "prepared"},
        # Figure 9's middle sizes: a row of 32^3 (128 KiB)
        {"name": "grid_32x32x3", "m": 1024, "factors": "32x32^3", "dtype": "float32", "call": "prepared"},
        # the largest: 4 GiB in, 4 GiB out
        {"name": "grid_32x32x4", "m": 1024, "factors": "32x32^4", "dtype": "float32", "call": "prepared"},
        # double precision with large factors on few rows, as in the Gaussian-process case study
        {"name": "gp_128x128x3_f64", "m": 16, "factors": "128x128^3", "dtype": "float64", "call": "prepared"},
        # double precision, Table 3 / Table 4 id 26: long rows of 16^6
        {"name": "gp_16x16x6_f64", "m": 16, "factors": "16x16^6", "dtype": "float64", "call": "prepared"},
        # rectangular factors that widen the rows sixteen times
        {"name": "widen_16x32x4", "m": 256, "factors": "16x32^4", "dtype": "float32", "call": "buffers"},
        # the backward direction of a Kron-Matmul with 64x64 factors (Figure 9)
        {"name": "gradient_64x64x3", "m": 1024, "factors": "64x64^3", "dtype": "float32", "call": "gradient"},
        # rows of odd length (5^8) and a row count that is no power of two
        {"name": "odd_5x5x8", "m": 1000, "factors": "5x5^8", "dtype": "float32", "call": "prepared"},
        # a grid of 100 points a side: factors that are no multiple of the matrix cores' blocks
        {"name": "grid_100x100x3", "m": 64, "factors": "100x100^3", "dtype": "float32", "call": "prepared"},
    ]


def _shapes(case):
    out = []
    for part in case["factors"].split(","):
        pq, _, n = part.partition("^")
        p, q = pq.split("x")
        out += [(int(p), int(q))] * int(n or 1)
    return out


def _text(shapes):
    return ",".join("%dx%d" % s for s in shapes)


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A problem of the same ranges: square chains and rectangular or mixed products, 1 to 4096 rows (odd counts
    among them), rows of up to 2^24 elements, at most 2^26 fp32 (2^25 fp64) elements in X or any intermediate."""
    while True:
        dtype = "float32" if rng.random() < 0.7 else "float64"
        most = 2 ** 26 if dtype == "float32" else 2 ** 25
        call = rng.choice(["prepared", "prepared", "plain", "buffers", "gradient"])
        m = _log_uniform(rng, 1, 4096)
        if rng.random() < 0.7:
            p = rng.choice([2, 3, 4, 5, 6, 7, 8, 8, 9, 10, 12, 14, 16, 16, 20, 24, 32, 32, 36, 48, 50, 64, 64, 80, 96, 100, 128, 128])
            q = p if rng.random() < 0.85 else rng.choice([max(1, p // 2), min(128, 2 * p)])
            deepest = max(1, int(math.log(2 ** 24) / math.log(p) + 1e-9))
            shapes = [(p, q)] * rng.randint(min(2, deepest), deepest)
        else:
            shapes = [(_log_uniform(rng, 2, 128), _log_uniform(rng, 2, 128)) for _ in range(rng.randint(2, 4))]
        k = widest = math.prod(p for p, _ in shapes)
        flops = 0
        for p, q in reversed(shapes):
            flops += 2 * m * k * q
            k = k // p * q
            widest = max(widest, k)
        if widest <= 2 ** 24 and 2 ** 6 <= m * widest <= most and flops <= 5e10:
            return {"m": m, "factors": _text(shapes), "dtype": dtype, "call": call}


def _inputs(case, seed):
    """The operand X (for a gradient: dY) and the factors of the product applied to it; entries of order one, with
    factors scaled so that the result stays of order one."""
    dtype = getattr(torch, case["dtype"])
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    shapes = _shapes(case)
    k = math.prod(p for p, _ in shapes)
    x = torch.randn((case["m"], k), dtype=dtype, device="cuda", generator=gen)
    fs = [torch.randn((p, q), dtype=dtype, device="cuda", generator=gen) / math.sqrt(p) for p, q in shapes]
    return x, fs


def prepare(case, seed):
    x, fs = _inputs(case, seed)
    state = {"call": case["call"], "x": x, "fs": fs}
    if case["call"] == "plain":
        return state
    transposed = case["call"] == "gradient"
    if transposed:
        # the forward product's factors: the transposes of those applied here
        state["fs"] = fs = [f.t().contiguous() for f in fs]
    p, q = zip(*_shapes(case))
    y = torch.empty((case["m"], math.prod(q)), dtype=x.dtype, device="cuda")
    need = km.workspace_size(case["m"], p, q, case["dtype"], transposed=transposed)
    ws = torch.empty(max(need, 1), dtype=torch.uint8, device="cuda")
    state["y"], state["ws"] = y, ws
    if case["call"] == "prepared":
        state["prepared"] = km.Prepared(x, fs, Y=y, workspace=ws)
    return state


def run(state):
    call = state["call"]
    if call == "prepared":
        return state["prepared"]()
    if call == "plain":
        return km.kronmatmul(state["x"], state["fs"])
    return km.kronmatmul(state["x"], state["fs"], Y=state["y"], workspace=state["ws"], transposed=call == "gradient")


def work(case):
    shapes = _shapes(case)
    size = 4 if case["dtype"] == "float32" else 8
    m = case["m"]
    k = math.prod(p for p, _ in shapes)
    elems, flops = m * k + sum(p * q for p, q in shapes), 0
    for p, q in reversed(shapes):
        flops += 2 * m * k * q
        k = k // p * q
    return {"bytes": size * (elems + m * k), "flops": flops}


def tolerance(case):
    # four times the largest distance from the 64-bit result over the listed cases (3.1e-7 at 100x100^3, 8.5e-16
    # at 128x128^3 in double precision): sums of the same products in another order differ by no more
    return {"rel": 1.3e-6} if case["dtype"] == "float32" else {"rel": 3.5e-15}


def exact(case, seed):
    """Algorithm 1 in plain 64-bit torch: contract the last index digit, put the new one in front."""
    x, fs = _inputs(case, seed)
    m = case["m"]
    z = x.double()
    del x
    for f in reversed(fs):
        p, q = f.shape
        s = z.numel() // (m * p)
        z = (z.reshape(m * s, p) @ f.double()).reshape(m, s, q).transpose(1, 2).contiguous().reshape(m, q * s)
    return z
