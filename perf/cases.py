"""The workloads by which this library's speed is judged: emulated GEMM calls through the public entry
points, on matrices that are resident on the GPU in column-major order (the layout of the C ABI).

A case is a dict of plain values:
  kind   "gemm"       real C = AB, FP64 or FP32 (gemm, or ozaki2_gemm / ozaki2_sgemm on a block of larger matrices)
         "complex"    complex C = AB, form "4m" (real embedding) or "3m" (three products per modulus)
         "certified"  gemm_certified: the planner picks the number of moduli, the error bound is checked after the run
         "batch"      gemm_batched_cm: independent problems of uneven sizes in one call
  prec   64 or 32; N: moduli; phi: exponent spread of the inputs
  m, n, k; or for a batch count, lo, hi, shape_seed (sizes log-uniform in [lo, hi])
  ld_extra  by how much each leading dimension exceeds the matrix (0: the matrices are whole buffers)

Inputs follow the paper's experiments (Section 5): (U - 0.5) exp(phi Z), each part of a complex matrix alike.
"""
from __future__ import annotations

import math
import random

import torch

import paper_2602_02549_amd as oz

DTYPE = {("real", 64): torch.float64, ("real", 32): torch.float32,
         ("complex", 64): torch.complex128, ("complex", 32): torch.complex64}


def _gemm(name, m, n, k, N, phi=0.5, prec=64, ld_extra=0):
    return {"name": name, "kind": "gemm", "prec": prec, "m": m, "n": n, "k": k, "N": N, "phi": phi,
            "ld_extra": ld_extra}


def _complex(name, m, n, k, N, form, phi=0.5, prec=64):
    return {"name": name, "kind": "complex", "prec": prec, "m": m, "n": n, "k": k, "N": N, "phi": phi,
            "form": form}


def listed():
    return [
        # The small configuration of the benchmark and the parity tests: many launches, little work.
        _gemm("dgemm_256", 256, 256, 256, 14),
        # The shape of the paper's experiments: a small output over a long inner dimension.
        _gemm("dgemm_128x128x8192", 128, 128, 8192, 16, phi=1.0),
        # A block of larger matrices with ragged sizes, as a factorisation's trailing update sees it.
        _gemm("dgemm_1000x700x1300_ld", 1000, 700, 1300, 15, ld_extra=24),
        # An ordinary square product.
        _gemm("dgemm_2048", 2048, 2048, 2048, 14),
        # Wide exponent spread, N as the bound asks for at 1e-15 (the benchmark's sweep).
        _gemm("dgemm_4096_phi2", 4096, 4096, 4096, 18, phi=2.0),
        # The headline product of the benchmark, N at which it matches native DGEMM's error.
        _gemm("dgemm_8192", 8192, 8192, 8192, 14),
        # Inner products over a very long dimension (Gram and overlap matrices), beyond the fused column pass.
        _gemm("dgemm_200x200x100000", 200, 200, 100000, 14),
        # FP32 emulation at the benchmark's size, N at which it matches native SGEMM.
        _gemm("sgemm_16384", 16384, 16384, 16384, 7, prec=32),
        # Complex products in both forms: ragged and ordinary through the real embedding, the benchmark's
        # size in three products.
        _complex("zgemm_1200x800x1500", 1200, 800, 1500, 14, "4m"),
        _complex("zgemm3m_4096", 4096, 4096, 4096, 15, "3m"),
        # A certified product: planner, run, certificate, and the host's decisions between them.
        {"name": "certified_4096", "kind": "certified", "prec": 64, "m": 4096, "n": 4096, "k": 4096,
         "phi": 1.0, "eps": 1e-14},
        # The benchmark's uneven batch.
        {"name": "batch_512", "kind": "batch", "prec": 64, "count": 512, "lo": 64, "hi": 2048,
         "shape_seed": 0, "N": 16, "phi": 1.0},
    ]


def _log_int(rng: random.Random, lo: int, hi: int) -> int:
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _moduli(rng: random.Random, prec: int) -> int:
    """FP64: mostly the N that matched error or a bound near 1e-15 asks for, now and then any; FP32: 6 to 9."""
    if prec == 32:
        return rng.randint(6, 9)
    return rng.randint(13, 18) if rng.random() < 0.75 else rng.randint(8, 49)


def draw(rng: random.Random):
    kind = rng.choice(["gemm"] * 5 + ["long"] + ["complex"] * 3 + ["certified"] + ["batch"] * 2)
    prec = 64 if rng.random() < 0.7 else 32
    phi = rng.choice([0.0, 0.5, 1.0, 2.0]) if prec == 64 else 0.5
    if kind == "long":   # small outputs over a long inner dimension
        return {"kind": "gemm", "prec": prec, "m": _log_int(rng, 48, 400), "n": _log_int(rng, 48, 400),
                "k": _log_int(rng, 8000, 260000), "N": _moduli(rng, prec), "phi": phi, "ld_extra": 0}
    if kind == "batch":
        lo = rng.choice([32, 64, 100])
        return {"kind": "batch", "prec": prec, "count": _log_int(rng, 8, 256), "lo": lo,
                "hi": _log_int(rng, 4 * lo, 2048), "shape_seed": rng.randrange(1 << 20),
                "N": _moduli(rng, prec), "phi": phi}
    if kind == "certified":
        return {"kind": "certified", "prec": 64, "m": _log_int(rng, 200, 4096), "n": _log_int(rng, 200, 4096),
                "k": _log_int(rng, 200, 4096), "phi": rng.choice([0.0, 0.5, 1.0]), "eps": 1e-14}
    top = 8192 if kind == "gemm" else 4096
    m, n, k = (_log_int(rng, 64, top) for _ in range(3))
    if rng.random() < 0.25:
        m = n = k
    if kind == "complex":
        return {"kind": "complex", "prec": prec, "m": m, "n": n, "k": k, "N": min(_moduli(rng, prec), 24),
                "phi": phi, "form": rng.choice(["4m", "3m"])}
    N = _moduli(rng, prec)
    if N > 20:           # the largest N on the largest sizes would cost more than any listed case
        m, n, k = min(m, 5000), min(n, 5000), min(k, 5000)
    return {"kind": "gemm", "prec": prec, "m": m, "n": n, "k": k, "N": N, "phi": phi,
            "ld_extra": rng.choice([0, 0, 1, 8, 37])}


def _shapes(case):
    """(m, n, k) of a batch's problems: the same for every seed."""
    rng = random.Random(case["shape_seed"])
    return [tuple(_log_int(rng, case["lo"], case["hi"]) for _ in range(3)) for _ in range(case["count"])]


def _entries(gen, shape, phi):
    u = torch.rand(shape, generator=gen, dtype=torch.float64, device="cuda")
    z = torch.randn(shape, generator=gen, dtype=torch.float64, device="cuda")
    return u.sub_(0.5).mul_(z.mul_(phi).exp_())


def _matrix(gen, rows, cols, case, what="real", ld_extra=0):
    """A logical rows x cols matrix, column-major (a transposed view); its columns are rows + ld_extra apart."""
    dtype = DTYPE[what, case["prec"]]
    X = _entries(gen, (cols, rows), case["phi"])
    if what == "complex":
        X = torch.complex(X, _entries(gen, (cols, rows), case["phi"]))
    buf = torch.zeros((cols, rows + ld_extra), dtype=dtype, device="cuda")
    buf[:, :rows] = X
    return buf[:, :rows].t() if ld_extra else buf.t()


def _pool(shapes, dtype):
    """One buffer for a batch's results and, per problem, its (n, m) part: a column-major m x n matrix."""
    starts, total = [], 0
    for m, n, _ in shapes:
        starts.append(total)
        total += (m * n + 63) // 64 * 64
    pool = torch.zeros(total, dtype=dtype, device="cuda")
    return pool, [pool[s:s + m * n].view(n, m) for s, (m, n, _) in zip(starts, shapes)]


def _operands(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    if case["kind"] == "batch":
        return [(_matrix(gen, m, k, case), _matrix(gen, k, n, case)) for m, n, k in _shapes(case)]
    what = "complex" if case["kind"] == "complex" else "real"
    ld = case.get("ld_extra", 0)
    return (_matrix(gen, case["m"], case["k"], case, what, ld),
            _matrix(gen, case["k"], case["n"], case, what, ld))


def prepare(case, seed):
    state = {"case": case}
    if case["kind"] == "batch":
        pairs, shapes = _operands(case, seed), _shapes(case)
        pool, C = _pool(shapes, DTYPE["real", case["prec"]])
        state.update(A=[A.t() for A, _ in pairs], B=[B.t() for _, B in pairs], shapes=shapes,
                     N=[case["N"]] * len(shapes), C=C, pool=pool)
        return state
    state["A"], state["B"] = _operands(case, seed)
    if case["kind"] == "gemm":
        state["C"] = torch.zeros((case["n"], case["m"] + case["ld_extra"]),
                                 dtype=DTYPE["real", case["prec"]], device="cuda")
    return state


def run(state):
    case, A, B = state["case"], state["A"], state["B"]
    if case["kind"] == "batch":
        oz.gemm_batched_cm(A, B, state["C"], state["shapes"], state["N"])
        return state["pool"]
    if case["kind"] == "certified":
        C, rc, N, ratio = oz.gemm_certified(A, B, case["eps"])
        return C, rc, N, ratio
    if case["kind"] == "complex":
        return oz.zgemm(A, B, case["N"], form=case["form"])
    C = state["C"]
    if case["ld_extra"] == 0:
        return oz.gemm(A, B, case["N"], out=C)
    oz.ozaki2_set_stream(torch.cuda.current_stream().cuda_stream)
    call = oz.ozaki2_gemm if case["prec"] == 64 else oz.ozaki2_sgemm
    rc = call(case["m"], case["n"], case["k"], A.data_ptr(), A.stride(1), B.data_ptr(), B.stride(1),
              C.data_ptr(), C.stride(0), case["N"])
    if rc != oz.OK:
        raise oz.Ozaki2Error("ozaki2_gemm", rc)
    return C[:, :case["m"]].t()


def work(case):
    """Each operand read once, C written once; INT8 operations of the scaling product and the residue products."""
    size = case["prec"] // 8
    if case["kind"] == "batch":
        shapes = _shapes(case)
        return {"bytes": sum(size * (m * k + k * n + m * n) for m, n, k in shapes),
                "flops": sum(2 * m * n * k * (case["N"] + 1) for m, n, k in shapes)}
    m, n, k = case["m"], case["n"], case["k"]
    data = size * (m * k + k * n + m * n)
    if case["kind"] == "complex":
        products = 4 * (case["N"] + 1) if case["form"] == "4m" else 3 * case["N"] + 1
        return {"bytes": 2 * data, "flops": 2 * m * n * k * products}
    if case["kind"] == "certified":   # about 15 moduli at 1e-14, the scaling product and one BF16 product
        return {"bytes": data, "flops": 2 * m * n * k * 17}
    return {"bytes": data, "flops": 2 * m * n * k * (case["N"] + 1)}


def exact(case, seed):
    """The products in FP64 (complex128) by torch."""
    wide = torch.complex128 if case["kind"] == "complex" else torch.float64
    if case["kind"] == "batch":
        pool, C = _pool(_shapes(case), wide)
        for c, (A, B) in zip(C, _operands(case, seed)):
            c.copy_(torch.matmul(A.to(wide), B.to(wide)).t())
        return pool
    A, B = _operands(case, seed)
    C = torch.matmul(A.to(wide), B.to(wide))
    if case["kind"] == "certified":
        return C, None, None, None
    return C
