"""The measured workloads: what a program built on this library has it do.

``listed()`` holds the fixed cases and ``draw(rng)`` gives further ones of the
same ranges; ``prepare`` makes what the program has in hand before a call (GPU
matrices, from a seed), ``run`` is one pass through the public Python entry
points, ``exact`` the same result from plain torch in 64 bits, and ``work``
the bytes and operations one pass cannot do without.

Kinds of case ("op"):

* ``invert``      FP64 inversion, the main call;
* ``spd``         FP64 inversion of a symmetric matrix (``invert_spd``);
* ``lu``          inversion through a block LU factorisation (``invert_lu``);
* ``mixed``       low-precision products refined by Newton steps;
* ``batch``       many independent requests in one call (``invert_batch``);
* ``gemm``        one block product with its fused epilogue (``gemm_cm``);
* ``gemm_int8``   one FP64-accurate product on INT8 matrix cores.

Matrices: "dd" is U(-1, 1) + n I, "gram" is B B^T / n + I with normal B, and
"spectrum" is Q diag(l) Q^T with l geometric over [1, kappa] and Q a cosine
basis with random signs and a random order of the eigenvalues.  "order" is the
memory order of the caller's tensors: "F" (the library's own) or "C" (what
torch makes by default).
"""
from __future__ import annotations

import math
import random

import torch

import paper_1801_04723_amd as spin

DEV = "cuda"
FP64_MODES = ("fp64", "fp64_sym")


def listed():
    return [
        # the smallest request of the serving mix, alone: one leaf, all latency
        {"name": "request_64", "op": "invert", "n": 64, "leaf": 64, "matrix": "dd", "order": "F"},
        # an ordinary torch matrix of an order that is no multiple of a tile
        {"name": "ragged_1000", "op": "invert", "n": 1000, "leaf": 128, "matrix": "spectrum", "kappa": 1e4,
         "order": "C"},
        # the headline workload: SPD, n = 8192, leaf 256
        {"name": "spd_matrix_8192", "op": "invert", "n": 8192, "leaf": 256, "matrix": "gram", "order": "F"},
        # the largest order of the leaf sweep, at its best leaf
        {"name": "sweep_16384", "op": "invert", "n": 16384, "leaf": 256, "matrix": "dd", "order": "F"},
        # the symmetric schedule on a covariance-like matrix
        {"name": "symmetric_4096", "op": "spd", "n": 4096, "leaf": 256, "matrix": "gram", "order": "F"},
        # the comparison method, at the leaf of its comparison
        {"name": "lu_2048", "op": "lu", "n": 2048, "leaf": 128, "matrix": "dd", "order": "F"},
        # a large mixed request of the serving mix
        {"name": "mixed_fp32_2048", "op": "mixed", "n": 2048, "leaf": 128, "matrix": "spectrum", "kappa": 1e3,
         "mode": "fp32", "steps": 2, "order": "F"},
        # BF16-split products, refined on INT8 matrix cores
        {"name": "mixed_bf16x3_int8_4096", "op": "mixed", "n": 4096, "leaf": 256, "matrix": "spectrum",
         "kappa": 1e3, "mode": "bf16x3_int8", "steps": 3, "order": "F"},
        # a burst of the serving mix: orders 64..1024, 70 % mixed, 30 % FP64
        {"name": "batch_24", "op": "batch", "count": 24, "n_min": 64, "n_max": 1024, "leaf": 128, "steps": 2,
         "shapes": 5, "order": "F"},
        # a Schur step of a caller's own blocks: D = C - A B, odd sizes
        {"name": "schur_ragged_fp64", "op": "gemm", "dtype": "fp64", "m": 1537, "n": 1001, "k": 777,
         "alpha": -1.0, "beta": 1.0},
        # the widest product of the split-BF16 path
        {"name": "product_bf16x3_4096", "op": "gemm", "dtype": "bf16x3", "m": 4096, "n": 4096, "k": 4096,
         "alpha": 1.0, "beta": 0.0},
        # a refinement residual I - A X on INT8 matrix cores
        {"name": "residual_int8_4096", "op": "gemm_int8", "m": 4096, "n": 4096, "k": 4096, "epilogue": 1},
    ]


def _size(rng, lo, hi):
    """An order spread over the logarithm of the range: a third odd or odd-sized, the rest multiples of 64 or 8."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    step = rng.choice((1, 8, 64))
    return int(min(hi, max(lo, step * round(v / step) if step > 1 else round(v))))


def draw(rng: random.Random):
    op = rng.choice(("invert", "invert", "invert", "spd", "lu", "mixed", "mixed", "batch", "gemm", "gemm", "gemm_int8"))
    order = rng.choice(("F", "C"))
    if op == "invert":
        n = _size(rng, 64, 8192)
        matrix = rng.choice(("dd", "gram", "spectrum"))
        return {"op": op, "n": n, "leaf": rng.choice((64, 128, 256, 512) if n > 256 else (32, 64, 128, 256)),
                "matrix": matrix, "kappa": 10.0 ** rng.uniform(1, 4), "order": order}
    if op == "spd":
        return {"op": op, "n": _size(rng, 128, 8192), "leaf": rng.choice((64, 128, 256)),
                "matrix": rng.choice(("gram", "spectrum")), "kappa": 10.0 ** rng.uniform(1, 4), "order": order}
    if op == "lu":
        return {"op": op, "n": _size(rng, 128, 4096), "leaf": rng.choice((64, 128)), "matrix": "dd",
                "order": order}
    if op == "mixed":
        mode = rng.choice(("fp32", "fp32", "bf16x3", "fp32_int8", "bf16x3_int8", "fp32_sym"))
        return {"op": op, "n": _size(rng, 128, 4096), "leaf": rng.choice((64, 128, 256)),
                "matrix": rng.choice(("dd", "spectrum")), "kappa": 10.0 ** rng.uniform(1, 3), "mode": mode,
                "steps": 3 if mode.startswith("bf16x3") else 2, "order": order}
    if op == "batch":
        return {"op": op, "count": rng.randrange(4, 33), "n_min": 64, "n_max": rng.choice((256, 512, 1024)),
                "leaf": rng.choice((64, 128)), "steps": 2, "shapes": rng.randrange(1 << 20), "order": order}
    if op == "gemm":
        alpha, beta = rng.choice(((1.0, 0.0), (-1.0, 0.0), (-1.0, 1.0)))
        return {"op": op, "dtype": rng.choice(("fp64", "fp64", "fp32", "bf16", "bf16x3")),
                "m": _size(rng, 64, 8192), "n": _size(rng, 64, 8192), "k": _size(rng, 64, 4096),
                "alpha": alpha, "beta": beta}
    m = _size(rng, 256, 4096)
    e = rng.choice((0, 1, 2))
    return {"op": op, "m": m, "n": m if e == 1 else _size(rng, 256, 4096), "k": _size(rng, 256, 4096), "epilogue": e}


# ------------------------------------------------------------------- inputs
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _rand(shape, g):
    return torch.rand(shape, generator=g, dtype=torch.float64, device=DEV) * 2.0 - 1.0


def _matrix(n, kind, kappa, seed):
    g = _gen(seed)
    if kind == "dd":
        a = _rand((n, n), g)
        a.diagonal().add_(float(n))
        return a
    if kind == "gram":
        b = torch.randn((n, n), generator=g, dtype=torch.float64, device=DEV)
        a = b @ b.t() / n
        a = 0.5 * (a + a.t())
        a.diagonal().add_(1.0)
        return a
    i = torch.arange(n, dtype=torch.float64, device=DEV)
    q = torch.cos(math.pi / n * (i[:, None] + 0.5) * i[None, :]) * math.sqrt(2.0 / n)
    q[:, 0] = math.sqrt(1.0 / n)
    q = q * torch.sign(_rand((n, 1), g) + 1e-300)
    lam = torch.pow(torch.tensor(float(kappa), dtype=torch.float64, device=DEV), i / max(n - 1, 1))
    lam = lam[torch.randperm(n, generator=g, device=DEV)]
    a = (q * lam[None, :]) @ q.t().contiguous()
    return 0.5 * (a + a.t())


def _ordered(a, order):
    return a.t().contiguous().t() if order == "F" else a.contiguous()


def _requests(case):
    """Orders, matrix kinds and modes of a batch: a function of the case alone."""
    r = random.Random(int(case["shapes"]))
    out = []
    for _ in range(int(case["count"])):
        raw = math.exp(r.uniform(math.log(case["n_min"]), math.log(case["n_max"])))
        n = max(64, min(int(64 * math.ceil(raw / 64)), int(case["n_max"])))
        kind = "dd" if r.random() < 0.5 else "spectrum"
        kappa = math.exp(r.uniform(math.log(10.0), math.log(1e4)))
        mode = "fp32" if r.random() < 0.7 else ("fp64" if kind == "dd" else "fp64_sym")
        out.append((n, kind, kappa, mode))
    return out


def _columns(rows, cols, dtype, g, scale=1.0):
    """A column-major rows x cols buffer (a contiguous cols x rows tensor)."""
    return (_rand((cols, rows), g) * scale).to(dtype)


def prepare(case, seed):
    op = case["op"]
    if op in ("invert", "spd", "lu", "mixed"):
        a = _matrix(case["n"], case["matrix"], case.get("kappa", 0.0), seed)
        return {"case": case, "a": _ordered(a, case["order"])}
    if op == "batch":
        reqs = _requests(case)
        mats = [_ordered(_matrix(n, kind, kappa, 1000003 * int(seed) + i), case["order"])
                for i, (n, kind, kappa, _) in enumerate(reqs)]
        return {"case": case, "mats": mats, "modes": [r[3] for r in reqs]}
    g = _gen(seed)
    m, n, k = case["m"], case["n"], case["k"]
    if op == "gemm":
        dt = torch.float64 if case["dtype"] == "fp64" else torch.float32
        st = {"case": case, "a": _columns(m, k, dt, g), "b": _columns(k, n, dt, g), "d": torch.empty((n, m), dtype=dt, device=DEV)}
        st["c"] = _columns(m, n, dt, g, math.sqrt(k)) if case["beta"] != 0.0 else None
        return st
    # operands of a refinement: a well-conditioned A and an approximate factor
    return {"case": case, "a": _columns(m, k, torch.float64, g), "b": _columns(k, n, torch.float64, g, 1.0 / math.sqrt(k)),
            "c": _columns(m, n, torch.float64, g) if case["epilogue"] == 2 else None,
            "d": torch.empty((n, m), dtype=torch.float64, device=DEV)}


# --------------------------------------------------------------------- pass
def run(state):
    case = state["case"]
    op = case["op"]
    if op == "invert":
        return spin.invert(state["a"], leaf=case["leaf"])
    if op == "spd":
        return spin.invert_spd(state["a"], leaf=case["leaf"])
    if op == "lu":
        return spin.invert_lu(state["a"], leaf=case["leaf"])
    if op == "mixed":
        return spin.invert_mixed(state["a"], leaf=case["leaf"], mode=case["mode"], ns_steps=case["steps"])
    if op == "batch":
        outs, info = spin.invert_batch(state["mats"], leaf=case["leaf"], modes=state["modes"], ns_steps=case["steps"])
        return {"outs": outs, "info": info}
    m, n, k = case["m"], case["n"], case["k"]
    a, b, c, d = state["a"], state["b"], state["c"], state["d"]
    if op == "gemm":
        spin.gemm_cm(m, n, k, case["alpha"], a, m, b, k, case["beta"], c, m, d, m, dtype=case["dtype"])
    else:
        spin.gemm_int8(m, n, k, a, m, b, k, case["epilogue"], c, m, d, m)
    return d


def exact(case, seed):
    state = prepare(case, seed)
    op = case["op"]
    if op in ("invert", "spd", "lu", "mixed"):
        return torch.linalg.inv(state["a"])
    if op == "batch":
        return {"outs": [torch.linalg.inv(a) for a in state["mats"]], "info": None}
    # the buffers are the column-major matrices' transposes: D^T = B^T A^T
    p = state["b"].double() @ state["a"].double()
    c = state["c"]
    if op == "gemm":
        d = case["alpha"] * p
        return d + case["beta"] * c.double() if c is not None else d
    if case["epilogue"] == 1:
        return torch.eye(case["m"], dtype=torch.float64, device=DEV) - p
    return p + c if case["epilogue"] == 2 else p


# --------------------------------------------------------------------- work
def work(case):
    op = case["op"]

    def inverse(n, mode, steps):
        """One inversion: the matrix in and out; 2 n^3 operations, n^3 for a
        symmetric matrix; a refinement step adds two products and the
        acceptance one more."""
        base = 1.0 if "sym" in mode else 2.0
        extra = 0.0 if mode in FP64_MODES else 2.0 * (2 * steps + 1)
        return 16.0 * n * n, (base + extra) * float(n) ** 3

    if op in ("invert", "lu"):
        b, f = inverse(case["n"], "fp64", 0)
    elif op == "spd":
        b, f = inverse(case["n"], "fp64_sym", 0)
    elif op == "mixed":
        b, f = inverse(case["n"], case["mode"], case["steps"])
    elif op == "batch":
        each = [inverse(n, mode, case["steps"]) for n, _, _, mode in _requests(case)]
        b, f = sum(x[0] for x in each), sum(x[1] for x in each)
    else:
        m, n, k = float(case["m"]), float(case["n"]), float(case["k"])
        size = 8.0 if op == "gemm_int8" or case["dtype"] == "fp64" else 4.0
        reads_c = case["epilogue"] == 2 if op == "gemm_int8" else case["beta"] != 0.0
        b, f = size * (m * k + k * n + (2.0 if reads_c else 1.0) * m * n), 2.0 * m * n * k
    return {"bytes": b, "flops": f}
