"""The workloads this library's speed is judged by: the calls its users make,
through the Python entry points, over the range of sizes they are made with.

* batched emulated products (``sgemm_emu_batched``): from one launch-bound
  batch of small products to one product that fills the device, whole and
  ragged sizes, narrow and wide ranges of magnitudes, shared right operands;
* the accumulate form with transposed operands (``sgemm_emu_batched_acc``):
  the products of a linear layer's backward pass, dX = dY W^T and
  dW = X^T dY added to what is there;
* the rule-built products (``householder_emu_batched``, ``givens_emu_batched``)
  and the scan (``sgemm_emu_scan``).

Inputs are drawn on the device from the seed; outputs go to buffers that the
state holds, as a program that makes the same call again and again holds them.
"""
import math

import torch

import paper_2308_15152_amd as emu

DEVICE = "cuda:0"


def listed():
    return [
        # the smallest call: sixteen 64^3 products, bound by the launch and
        # the host path (per-block products inside a larger solver step)
        gemm("gemm_64", 16, 64, 64, 64),
        # a large batch of one-tile products, bound by memory
        gemm("gemm_128", 4096, 128, 128, 128),
        # a batch of 256^3 products whose entries span 30 binades
        gemm("gemm_256e", 1024, 256, 256, 256, dist="uniform_exp"),
        # one large product, bound by the matrix units
        gemm("gemm_8192", 1, 8192, 8192, 8192),
        # an ordinary single product whose sizes fill no whole tiles
        gemm("gemm_1100", 1, 1100, 1500, 2000),
        # a few products of odd sizes: packed rows of odd length, so no row
        # but the first is aligned
        gemm("gemm_odd", 8, 1001, 999, 1003),
        # weight gradients of many small blocks, D = A^T B + C
        acc("acc_128_tn", 4096, 128, 128, 128, True, False),
        # input gradient of one wide layer, D = A B^T + C
        acc("acc_4096_nt", 1, 4096, 4096, 4096, False, True),
        # reflectors applied to a large batch of 64 x 64 blocks
        {"name": "householder_64", "kind": "householder", "batch": 262144, "ncols": 64},
        # one rotation plane over a large batch of 64 x 64 blocks
        {"name": "givens_64", "kind": "givens", "batch": 262144, "ncols": 64, "i": 5, "j": 37},
        # many rows of ordinary length (running sums over a feature axis)
        {"name": "scan_2048", "kind": "scan", "rows": 131072, "len": 2048},
        # a few long rows (running sums over a signal or a histogram)
        {"name": "scan_1m", "kind": "scan", "rows": 32, "len": 1000000},
    ]


def gemm(name, batch, m, n, k, dist="uniform", shared_b=False):
    c = {"kind": "gemm", "batch": batch, "m": m, "n": n, "k": k, "dist": dist,
         "shared_b": shared_b}
    return dict(c, name=name) if name else c


def acc(name, batch, m, n, k, ta, tb, in_place=False):
    c = {"kind": "acc", "batch": batch, "m": m, "n": n, "k": k, "ta": ta, "tb": tb,
         "in_place": in_place}
    return dict(c, name=name) if name else c


# A drawn case moves at most this many bytes and runs at most this many
# emulated flops (the largest listed ones: 8.7 GB and 1.1 Tflop).
MAX_BYTES = 4e9
MAX_FLOPS = 2.6e11


def log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def size(rng, lo, hi):
    """A size of [lo, hi], even over its logarithm: odd or any (half of the
    draws), or a multiple of 4, 32 or 128."""
    grain = rng.choice([1, 1, 1, 4, 32, 128])
    v = log_int(rng, lo, hi)
    return max(lo, v - v % grain) if grain > 1 else v


def draw(rng):
    kind = rng.choice(["gemm", "gemm", "gemm", "acc", "acc", "householder", "givens", "scan"])
    if kind in ("gemm", "acc"):
        m, n, k = (size(rng, 32, 4096) for _ in range(3))
        per_flops = 2.0 * m * n * k
        per_bytes = 4.0 * (m * k + k * n + 2 * m * n)
        most = min(4096, MAX_FLOPS / per_flops, MAX_BYTES / per_bytes)
        batch = log_int(rng, 1, max(1.0, most))
        if kind == "gemm":
            return gemm(None, batch, m, n, k, dist=rng.choice(["uniform", "uniform_exp"]),
                        shared_b=rng.random() < 0.25)
        return acc(None, batch, m, n, k, rng.random() < 0.5, rng.random() < 0.5,
                   in_place=rng.random() < 0.5)
    if kind in ("householder", "givens"):
        ncols = size(rng, 16, 512)
        batch = log_int(rng, 64, MAX_BYTES / (4.0 * 2 * 64 * ncols))
        if kind == "householder":
            return {"kind": kind, "batch": batch, "ncols": ncols}
        i, j = rng.sample(range(64), 2)
        return {"kind": kind, "batch": batch, "ncols": ncols, "i": i, "j": j}
    length = size(rng, 128, 1000000)
    rows = log_int(rng, max(1, 2 ** 17 // length), min(131072, 2 ** 28 // length))
    return {"kind": "scan", "rows": rows, "len": length}


def uniform(shape, g):
    """uniform(-1, 1) on the 2^-23 grid."""
    return torch.rand(shape, generator=g, dtype=torch.float32, device=DEVICE).mul_(2.0).sub_(1.0)


def uniform_exp(shape, g):
    """uniform(-1, 1) times 2^e, e a whole number of [-15, 15] per entry."""
    u = uniform(shape, g)
    e = torch.randint(-15, 16, shape, generator=g, dtype=torch.int32, device=DEVICE)
    return torch.ldexp(u, e.to(torch.float32))


def inputs(case, seed):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(seed)
    kind = case["kind"]
    if kind == "gemm":
        entries = uniform if case["dist"] == "uniform" else uniform_exp
        A = entries((case["batch"], case["m"], case["k"]), g)
        B = entries((case["k"], case["n"]) if case["shared_b"]
                    else (case["batch"], case["k"], case["n"]), g)
        return {"A": A, "B": B}
    if kind == "acc":
        b, m, n, k = case["batch"], case["m"], case["n"], case["k"]
        return {"A": uniform((b, k, m) if case["ta"] else (b, m, k), g),
                "B": uniform((b, n, k) if case["tb"] else (b, k, n), g),
                "C": uniform((b, m, n), g)}
    if kind == "householder":
        u = torch.randn((case["batch"], 64), generator=g, dtype=torch.float32, device=DEVICE)
        u /= torch.linalg.vector_norm(u, dim=1, keepdim=True)
        return {"u": u, "B": uniform((case["batch"], 64, case["ncols"]), g)}
    if kind == "givens":
        t = torch.rand((case["batch"],), generator=g, dtype=torch.float64, device=DEVICE)
        t *= 2.0 * math.pi
        return {"c": t.cos().float(), "s": t.sin().float(),
                "B": uniform((case["batch"], 64, case["ncols"]), g)}
    return {"X": uniform((case["rows"], case["len"]), g)}


def prepare(case, seed):
    state = inputs(case, seed)
    state["case"] = case
    kind = case["kind"]
    if kind in ("gemm", "acc"):
        out = (case["batch"], case["m"], case["n"])
    elif kind == "scan":
        out = (case["rows"], case["len"])
    else:
        out = (case["batch"], 64, case["ncols"])
    state["out"] = torch.empty(out, dtype=torch.float32, device=DEVICE)
    return state


def run(state):
    case, out = state["case"], state["out"]
    kind = case["kind"]
    if kind == "gemm":
        return emu.sgemm_emu_batched(state["A"], state["B"], out)
    if kind == "acc":
        addend = state["C"]
        if case["in_place"]:  # a gradient buffer that starts from C and is added to
            addend = out.copy_(addend)
        return emu.sgemm_emu_batched_acc(state["A"], state["B"], addend, out,
                                         op_a=emu.OP_T if case["ta"] else emu.OP_N,
                                         op_b=emu.OP_T if case["tb"] else emu.OP_N)
    if kind == "householder":
        return emu.householder_emu_batched(state["u"], state["B"], out)
    if kind == "givens":
        return emu.givens_emu_batched(case["i"], case["j"], state["c"], state["s"], state["B"],
                                      out)
    return emu.sgemm_emu_scan(state["X"], out)


def work(case):
    kind = case["kind"]
    if kind in ("gemm", "acc"):
        b, m, n, k = case["batch"], case["m"], case["n"], case["k"]
        shared = case.get("shared_b", False)
        addend = m * n * (3 if case.get("in_place") else 1) if kind == "acc" else 0
        values = b * (m * k + m * n + addend) + k * n * (1 if shared else b)
        # the method's three matrix products for each emulated one
        return {"bytes": 4 * values, "flops": 3 * 2 * b * m * n * k}
    if kind == "scan":
        return {"bytes": 8 * case["rows"] * case["len"], "flops": case["rows"] * case["len"]}
    b, nc = case["batch"], case["ncols"]
    if kind == "householder":
        # u and B read, C written; C = B - 2 u (u^T B)
        return {"bytes": 4 * b * (64 + 2 * 64 * nc), "flops": b * 4 * 64 * nc}
    return {"bytes": 4 * b * (2 + 2 * 64 * nc), "flops": b * 6 * nc}


def tolerance(case):
    """Four times the 2-norm error against exact() that was measured: 7.5e-8
    for k = 64, 9.1e-8 for 128, 2.9e-7 for 2000, 5.8e-7 for 8192 (the split's
    two roundings, and FP32 sums whose error grows with the square root of
    their length); 8.1e-8 for reflectors, 2.3e-8 for rotations; 7.6e-8 for
    running sums of 2048 values, 4.4e-7 to 5.4e-7 of 1000000.  An output may be
    off by more: twelve times that against the root mean square."""
    kind = case["kind"]
    if kind in ("gemm", "acc"):
        rel = 4 * (5e-8 + 6.5e-9 * math.sqrt(case["k"]))
    elif kind == "scan":
        rel = 4 * (7e-8 + 5e-10 * math.sqrt(case["len"]))
    else:
        rel = 4 * (8e-8 if kind == "householder" else 2.5e-8)
    return {"rel": rel, "max": 12 * rel}


def exact(case, seed):
    x = inputs(case, seed)
    kind = case["kind"]
    if kind == "gemm":
        A, B = x["A"].double(), x["B"].double()
        return torch.matmul(A, B)
    if kind == "acc":
        A = (x["A"].mT if case["ta"] else x["A"]).double().contiguous()
        B = (x["B"].mT if case["tb"] else x["B"]).double().contiguous()
        return torch.matmul(A, B).add_(x["C"])
    if kind == "householder":
        u, B = x["u"].double(), x["B"].double()
        return B.sub_(torch.bmm(u[:, :, None], torch.bmm(u[:, None, :], B)), alpha=2.0)
    if kind == "givens":
        c, s = x["c"].double()[:, None], x["s"].double()[:, None]
        out = x["B"].double()
        bi, bj = out[:, case["i"]].clone(), out[:, case["j"]].clone()
        out[:, case["i"]] = c * bi - s * bj
        out[:, case["j"]] = s * bi + c * bj
        return out
    return x["X"].double().cumsum(dim=1)
