"""The work this library is measured on: one pass of each public entry point over the sizes its users bring.

A case is a dict of plain values:

* ``gemm``     one ``gemm`` call: M, N, K, mode, preconverted operands or FP32 ones, beta
* ``batched``  one ``gemm_batched`` call on `count` equal problems
* ``grouped``  one run of a ``GroupedPlan`` over `count` uneven problems, M, N, K log-uniform in [16, 512]
* ``solve``    one ``solve_ir`` call: an FP64 system solved by refining a mixed-precision factorisation
* ``serve``    a burst of requests through a ``Server``, M, N, K log-uniform in [32, 4096], four modes, then a drain

``sizes`` seeds the problem sizes of a grouped or served case (the amount of work belongs to the case); the seed given
to ``prepare`` draws the values only.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

import paper_1803_04014_amd as mfg

DEV = "cuda"
PLANES = {"f16": (1, 1), "bf16": (1, 1), "refine_a": (2, 1), "split3": (2, 2), "split4": (2, 2), "bf16_split3": (2, 2)}
SERVED = ("f16", "bf16", "split3", "fp8")


def listed():
    return [
        # the paper's headline: one large half-precision GEMM, C = A B + C
        gemm("f16_8192", 8192, 8192, 8192, "f16", pre=True, beta=1.0),
        # the smallest single calls, where latency counts
        gemm("bf16_256", 256, 256, 256, "bf16", pre=True),
        # a request of no particular size, refined to FP32 accuracy, operands as the user has them
        gemm("split3_ragged", 777, 1234, 1999, "split3"),
        # the refined product at an ordinary size, from FP32 (both operands split in the call)
        gemm("split3_4096", 4096, 4096, 4096, "split3"),
        # the single-precision GEMM the refinement is compared with
        gemm("f32_2048", 2048, 2048, 2048, "f32"),
        # the 8-bit format, quantised in the call
        gemm("fp8_4096", 4096, 4096, 4096, "fp8"),
        # the paper's batched study: very many 16 x 16 x 16 problems
        {"name": "batched_16", "what": "batched", "count": 65536, "M": 16, "N": 16, "K": 16, "mode": "f16"},
        # the batched study's larger problems
        {"name": "batched_64", "what": "batched", "count": 16384, "M": 64, "N": 64, "K": 64, "mode": "f16"},
        # thousands of uneven problems on half-precision operands, replayed as a graph
        {"name": "grouped_f16", "what": "grouped", "count": 4096, "mode": "f16", "fp32": False, "graph": True, "sizes": 6},
        # the same problems refined, from FP32 operands
        {"name": "grouped_split3_fp32", "what": "grouped", "count": 4096, "mode": "split3", "fp32": True, "graph": False,
         "sizes": 6},
        # a linear system solved to FP64 accuracy on a refined factorisation
        {"name": "solve_2048", "what": "solve", "n": 2048, "nrhs": 1, "mode": "split3"},
        # a burst of mixed requests through the server
        {"name": "serve_64", "what": "serve", "count": 64, "sizes": 11},
    ]


def gemm(name, M, N, K, mode, pre=False, beta=0.0):
    c = {"what": "gemm", "M": M, "N": N, "K": K, "mode": mode, "pre": pre, "beta": beta}
    return {"name": name, **c} if name else c


def draw(rng):
    what = rng.choices(["gemm", "batched", "grouped", "solve", "serve"], [10, 3, 3, 2, 2])[0]
    if what == "gemm":
        mode = rng.choice(["f16", "bf16", "refine_a", "split3", "split4", "bf16_split3", "bf16_split6", "f32", "fp8"])
        dims = [log_uniform(rng, 32, 4096) for _ in range(3)]
        if rng.random() < 0.5:  # sizes somebody chose: multiples of 64
            dims = [max(64, (d + 32) // 64 * 64) for d in dims]
        pre = mode not in ("f32", "bf16_split6") and rng.random() < 0.5
        return gemm(None, *dims, mode, pre=pre, beta=rng.choice([0.0, 0.0, 1.0]))
    if what == "batched":
        M, N, K = (rng.randint(8, 64) for _ in range(3))
        if rng.random() < 0.5:
            M = N = K = rng.choice([8, 16, 32, 48, 64])
        each = 4 * (M * K + K * N + M * N)
        return {"what": "batched", "count": min(log_uniform(rng, 64, 65536), 800_000_000 // each), "M": M, "N": N, "K": K,
                "mode": rng.choice(["f16", "bf16", "f32", "split3"])}
    if what == "grouped":
        return {"what": "grouped", "count": log_uniform(rng, 64, 4096), "mode": rng.choice(sorted(PLANES)),
                "fp32": rng.random() < 0.5, "graph": rng.random() < 0.5, "sizes": rng.randrange(1 << 30)}
    if what == "solve":
        return {"what": "solve", "n": log_uniform(rng, 64, 2048), "nrhs": rng.choice([1, 1, 3, 16]),
                "mode": rng.choice(["f32", "split3", "bf16_split3"])}
    return {"what": "serve", "count": log_uniform(rng, 8, 64), "sizes": rng.randrange(1 << 30)}


def log_uniform(rng, lo, hi):
    return min(hi, max(lo, round(math.exp(rng.uniform(math.log(lo), math.log(hi))))))


def up(x, m):
    return (x + m - 1) // m * m


def sizes_of(case):
    """(M, N, K) of every problem of a grouped or served case."""
    rng = random.Random(case["sizes"])
    lo, hi = (16, 512) if case["what"] == "grouped" else (32, 4096)
    return [tuple(log_uniform(rng, lo, hi) for _ in range(3)) for _ in range(case["count"])]


def modes_of(case):
    rng = random.Random(case["sizes"] + 1)
    return [rng.choice(SERVED) for _ in range(case["count"])]


class Values:
    """Device tensors drawn in order from one seed."""

    def __init__(self, seed):
        self.g = torch.Generator(device=DEV)
        self.g.manual_seed(seed)

    def uniform(self, *shape):
        return torch.rand(shape, device=DEV, generator=self.g).mul_(2).sub_(1)

    def normal(self, *shape, dtype=torch.float32):
        return torch.randn(shape, device=DEV, generator=self.g, dtype=dtype)


# ------------------------------------------------------------------ inputs
def gemm_values(case, seed):
    v = Values(seed)
    return v.uniform(case["M"], case["K"]), v.uniform(case["K"], case["N"]), v.uniform(case["M"], case["N"])


def preconverted(X, mode):
    """X in the mode's storage form, as a 2-D tensor whose row stride is its leading dimension."""
    rows, cols = X.shape
    ld = up(cols, 16 if mode == "fp8" else 8)
    buf = torch.zeros(mfg.convert_bytes(rows, cols, ld, mode), dtype=torch.uint8, device=DEV)
    mfg.convert(X, buf, ld, mode)
    if mode == "fp8":
        return buf.as_strided((rows, cols), (ld, 1))
    return buf.view(torch.int16).as_strided((rows, cols), (ld, 1))


def batched_values(case, seed):
    v, n = Values(seed), case["count"]
    A, B = v.uniform(n, case["M"], case["K"]), v.uniform(n, case["K"], case["N"])
    t = {"f16": torch.float16, "bf16": torch.bfloat16}.get(case["mode"], torch.float32)
    return A.to(t), B.to(t)


class Packed:
    """Matrices one after the other in one tensor, each from an offset that is a multiple of 64 elements."""

    def __init__(self, shapes, ld_multiple=1):
        self.at, n = [], 0
        for rows, cols in shapes:
            ld = up(cols, ld_multiple)
            self.at.append((rows, cols, ld, n))
            n += up(rows * ld, 64)
        self.size = n

    def views(self, pool):
        return [pool.as_strided((r, c), (ld, 1), at) for r, c, ld, at in self.at]


def grouped_values(case, seed):
    """Operands of every problem as views of two pools: FP32 matrices contiguous, half-precision rows 16-byte aligned."""
    dims, ld = sizes_of(case), 1 if case["fp32"] else 8
    pa, pb = Packed([(m, k) for m, n, k in dims], ld), Packed([(k, n) for m, n, k in dims], ld)
    v = Values(seed)
    return pa, pb, v.uniform(pa.size), v.uniform(pb.size)


def solve_values(case, seed):
    v, n = Values(seed), case["n"]
    A = v.normal(n, n, dtype=torch.float64)
    A.diagonal().add_(2.0 * math.sqrt(n))
    return A, v.normal(n, case["nrhs"], dtype=torch.float64)


def serve_values(case, seed):
    v = Values(seed)
    dims = sizes_of(case)
    top = [max(d[i] for d in dims) for i in range(3)]
    return v.normal(top[0], top[2]), v.normal(top[2], top[1])


# ------------------------------------------------------------- prepare, run
def prepare(case, seed):
    s, what = {"case": case}, case["what"]
    if what == "gemm":
        A, B, C = gemm_values(case, seed)
        if case["pre"]:
            A, B = preconverted(A, case["mode"]), preconverted(B, case["mode"])
        s.update(A=A, B=B, C=C)
    elif what == "batched":
        A, B = batched_values(case, seed)
        s.update(A=A, B=B, C=torch.zeros(case["count"], case["M"], case["N"], device=DEV))
    elif what == "grouped":
        pa, pb, A, B = grouped_values(case, seed)
        mode, dims = case["mode"], sizes_of(case)
        if case["fp32"]:
            As, Bs = pa.views(A), pb.views(B)
        elif mode in ("f16", "bf16"):
            t = torch.float16 if mode == "f16" else torch.bfloat16
            As, Bs = pa.views(A.to(t)), pb.views(B.to(t))
        else:
            As = [preconverted(X, mode) for X in pa.views(A)]
            Bs = [preconverted(X, mode if PLANES[mode][1] == 2 else "f16") for X in pb.views(B)]
        pc = Packed([(m, n) for m, n, k in dims])
        s["C"] = torch.zeros(pc.size, device=DEV)
        s["plan"] = mfg.GroupedPlan(list(zip(As, Bs, pc.views(s["C"]))), mode, fp32_in=case["fp32"])
    elif what == "solve":
        A, B = solve_values(case, seed)
        s.update(A=A, B=B, X=torch.zeros_like(B))
    else:
        A, B = serve_values(case, seed)
        dims, modes = sizes_of(case), modes_of(case)
        s["C"], s["requests"] = {}, []
        for mode in SERVED:
            mine = [d for d, m in zip(dims, modes) if m == mode]
            if not mine:
                continue
            pc = Packed([(m, n) for m, n, k in mine])
            s["C"][mode] = torch.zeros(pc.size, device=DEV)
            s["requests"] += [(A[:m, :k], B[:k, :n], C, mode) for (m, n, k), C in zip(mine, pc.views(s["C"][mode]))]
        random.Random(case["sizes"]).shuffle(s["requests"])
        torch.cuda.synchronize()  # the server reads the operands on streams of its own
        s["server"] = mfg.Server(hbm_budget_bytes=8 << 30, slots=4, device=torch.cuda.current_device(), max_group=16)
    return s


def run(s):
    case = s["case"]
    what = case["what"]
    if what == "gemm":
        mfg.gemm(s["A"], s["B"], s["C"], 1.0, case["beta"], mode=case["mode"], preconverted=case["pre"])
        return s["C"]
    if what == "batched":
        mfg.gemm_batched(s["A"], s["B"], s["C"], mode=case["mode"])
        return s["C"]
    if what == "grouped":
        (s["plan"].graph_launch if case["graph"] else s["plan"].run)(1.0, 0.0)
        return s["C"]
    if what == "solve":
        mfg.solve_ir(s["A"], s["B"], s["X"], mode=case["mode"])
        return s["X"]
    tickets = [s["server"].submit(*r) for r in s["requests"]]
    s["server"].drain()
    for t in tickets:
        s["server"].poll(t)
    return s["C"]


# -------------------------------------------------------------------- work
def operand_bytes(mode, rows, cols, side, pre):
    """Bytes of one operand as the call receives it."""
    if not pre:
        return 4 * rows * cols
    return rows * cols * (1 if mode == "fp8" else 2 * PLANES[mode][side])


def work(case):
    what = case["what"]
    if what == "gemm":
        M, N, K, mode, pre = case["M"], case["N"], case["K"], case["mode"], case["pre"]
        return {"bytes": operand_bytes(mode, M, K, 0, pre) + operand_bytes(mode, K, N, 1, pre) +
                M * N * (8 if case["beta"] else 4), "flops": 2 * M * N * K}
    if what == "batched":
        n, M, N, K = case["count"], case["M"], case["N"], case["K"]
        e = 2 if case["mode"] in ("f16", "bf16") else 4
        return {"bytes": n * (e * (M * K + K * N) + 4 * M * N), "flops": 2 * n * M * N * K}
    if what == "solve":  # the factorisation, and reading the FP64 system once
        n = case["n"]
        return {"bytes": 8 * n * n + 16 * n * case["nrhs"], "flops": 2 * n ** 3 // 3 + 2 * n * n * case["nrhs"]}
    dims, pre = sizes_of(case), what == "grouped" and not case["fp32"]
    mode = case.get("mode")
    return {"bytes": sum(operand_bytes(mode, m, k, 0, pre) + operand_bytes(mode, k, n, 1, pre) + 4 * m * n
                         for m, n, k in dims), "flops": sum(2 * m * n * k for m, n, k in dims)}


# ------------------------------------------------------------------- exact
def operand64(X, mode):
    """What the mode multiplies, in 64 bits: rounded to the half-precision format, else (refined, 8-bit and FP32) X itself."""
    if mode in ("f16", "bf16"):
        X = X.to(torch.float16 if mode == "f16" else torch.bfloat16)
    return X.double()


def exact(case, seed):
    what = case["what"]
    if what == "gemm":
        A, B, C = gemm_values(case, seed)
        return operand64(A, case["mode"]) @ operand64(B, case["mode"]) + case["beta"] * C.double()
    if what == "batched":
        A, B = batched_values(case, seed)
        return torch.bmm(A.double(), B.double())
    if what == "grouped":
        pa, pb, A, B = grouped_values(case, seed)
        dims, mode = sizes_of(case), case["mode"]
        pc = Packed([(m, n) for m, n, k in dims])
        C = torch.zeros(pc.size, device=DEV, dtype=torch.float64)
        for a, b, c in zip(pa.views(operand64(A, mode)), pb.views(operand64(B, mode)), pc.views(C)):
            torch.mm(a, b, out=c)
        return C
    if what == "solve":
        A, B = solve_values(case, seed)
        return torch.from_numpy(np.linalg.solve(A.cpu().numpy(), B.cpu().numpy()))
    A, B = serve_values(case, seed)
    dims, modes, out = sizes_of(case), modes_of(case), {}
    for mode in SERVED:
        mine = [d for d, m in zip(dims, modes) if m == mode]
        if not mine:
            continue
        pc = Packed([(m, n) for m, n, k in mine])
        out[mode] = torch.zeros(pc.size, device=DEV, dtype=torch.float64)
        for (m, n, k), c in zip(mine, pc.views(out[mode])):
            torch.mm(operand64(A[:m, :k], mode), operand64(B[:k, :n], mode), out=c)
    return out
