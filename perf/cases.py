"""Performance cases of the spx library: what its users run, through
paper_2006_14290_amd.spx, over the sizes that they run it at.

A case is a dict of plain values:
  kind    spmv | convert | transpose | solve | ir | batch
  matrix  poisson2d (5-point, N x N), stencil7 / aniso7 / convdiff7 (7-point,
          N^3), stencil27 (27-point pattern, N^3, random values), zipf (Zipf(1.5)
          row lengths clipped at 10,000, uniform columns, N rows), spd (random
          symmetric diagonally dominant, N rows, about 16 entries per row)
  N, fmt, dtype, ...   the size, the storage format and value type, and each
          kind's own options.

The matrices are the ones of the tests and of the benchmark; they are made
with torch on the device, since they are made often.
"""
import math
import random

import numpy as np
import torch

from paper_2006_14290_amd import spx, synth

DEV = "cuda"
FMT = {"csr": spx.CSR, "coo": spx.COO, "ell": spx.ELL, "hyb": spx.HYB, "sellp": spx.SELLP}
DT = {"f64": spx.F64, "f32": spx.F32, "f16": spx.F16}
SIZE = {"f64": 8, "f32": 4, "f16": 2}


def listed():
    return [
        # one product of a small system, as in a time step that calls the
        # library once: the cost of a call
        {"name": "spmv_csr_f64_poisson2d_64", "kind": "spmv", "matrix": "poisson2d", "N": 64, "fmt": "csr",
         "dtype": "f64", "beta": 0.0},
        # the benchmark's product: a finite-element-like stencil, float64
        {"name": "spmv_csr_f64_stencil27_100", "kind": "spmv", "matrix": "stencil27", "N": 100, "fmt": "csr",
         "dtype": "f64", "beta": 0.0},
        # the product inside mixed-precision refinement: binary16 values,
        # float32 vectors, short rows
        {"name": "spmv_csr_f16_stencil7_192", "kind": "spmv", "matrix": "stencil7", "N": 192, "fmt": "csr",
         "dtype": "f16", "beta": 0.0},
        # single precision in the sliced format, an odd size, with an
        # accumulated result (y = A x + beta y)
        {"name": "spmv_sellp_f32_stencil27_101", "kind": "spmv", "matrix": "stencil27", "N": 101, "fmt": "sellp",
         "dtype": "f32", "beta": -0.5},
        # a graph-like matrix: skewed rows, random columns, the hybrid format
        {"name": "spmv_hyb_f64_zipf_1000000", "kind": "spmv", "matrix": "zipf", "N": 1_000_000, "fmt": "hyb",
         "dtype": "f64", "beta": 0.0},
        # a matrix assembled in CSR, moved to ELL for its products and back
        {"name": "convert_ell_f64_stencil27_100", "kind": "convert", "matrix": "stencil27", "N": 100, "fmt": "ell",
         "dtype": "f64"},
        # A^T of a nonsymmetric operator
        {"name": "transpose_f64_convdiff7_128", "kind": "transpose", "matrix": "convdiff7", "N": 128,
         "dtype": "f64"},
        # one small solve at a time: latency
        {"name": "cg_csr_poisson2d_64", "kind": "solve", "solver": "cg", "precond": 0, "matrix": "poisson2d", "N": 64,
         "fmt": "csr"},
        # the full-size symmetric solve
        {"name": "cg_jacobi_csr_aniso7_128", "kind": "solve", "solver": "cg", "precond": 1, "matrix": "aniso7",
         "N": 128, "fmt": "csr"},
        # the full-size nonsymmetric solve
        {"name": "gmres_jacobi_csr_convdiff7_128", "kind": "solve", "solver": "gmres", "precond": 1,
         "matrix": "convdiff7", "N": 128, "fmt": "csr"},
        # mixed-precision refinement around binary16 values
        {"name": "ir_csr_f16_stencil7_128", "kind": "ir", "matrix": "stencil7", "N": 128, "fmt": "csr",
         "dtype": "f16"},
        # many independent systems of mixed size at once, as the solve
        # server advances them
        {"name": "batch_mix_32", "kind": "batch", "count": 32, "mix": 1},
    ]


def _odd(rng, lo, hi):
    """A size spread over the logarithm of [lo, hi]."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["spmv", "spmv", "spmv", "convert", "transpose", "solve", "solve", "ir", "batch"])
    if kind == "spmv":
        m = rng.choice(["poisson2d", "stencil7", "stencil27", "zipf", "spd"])
        lo, hi = {"poisson2d": (33, 1500), "stencil7": (16, 190), "stencil27": (12, 110), "zipf": (5000, 900_000),
                  "spd": (1000, 900_000)}[m]
        # ELL stores every row at the length of the longest: for even rows only
        fmt = rng.choice(["csr", "csr", "coo", "hyb"] + ([] if m == "zipf" else ["ell", "sellp"]))
        return {"kind": kind, "matrix": m, "N": _odd(rng, lo, hi), "fmt": fmt,
                "dtype": rng.choice(["f64", "f64", "f32", "f16"]), "beta": rng.choice([0.0, 0.0, 0.0, -0.5])}
    if kind == "convert":
        m = rng.choice(["poisson2d", "stencil7", "stencil27", "spd"])
        lo, hi = {"poisson2d": (33, 1500), "stencil7": (16, 150), "stencil27": (12, 99), "spd": (1000, 900_000)}[m]
        return {"kind": kind, "matrix": m, "N": _odd(rng, lo, hi), "fmt": rng.choice(["coo", "ell", "hyb", "sellp"]),
                "dtype": rng.choice(["f64", "f64", "f32", "f16"])}
    if kind == "transpose":
        m = rng.choice(["poisson2d", "convdiff7", "stencil27", "spd", "zipf"])
        lo, hi = {"poisson2d": (33, 1500), "convdiff7": (16, 128), "stencil27": (12, 80), "spd": (1000, 800_000),
                  "zipf": (5000, 100_000)}[m]
        return {"kind": kind, "matrix": m, "N": _odd(rng, lo, hi), "dtype": rng.choice(["f64", "f64", "f32", "f16"])}
    if kind == "solve":
        solver = rng.choice(["cg", "cg", "bicgstab", "gmres", "bicg", "pipecg"])
        if solver in ("cg", "pipecg"):
            m, lo, hi = rng.choice([("poisson2d", 33, 400), ("aniso7", 17, 120), ("stencil7", 17, 140),
                                    ("spd", 1000, 500_000)])
        else:
            m, lo, hi = "convdiff7", 17, 120
        fmt = "csr" if solver == "bicg" else rng.choice(["csr", "csr", "csr", "ell", "sellp"])
        return {"kind": kind, "solver": solver, "precond": rng.choice([0, 1]), "matrix": m, "N": _odd(rng, lo, hi),
                "fmt": fmt}
    if kind == "ir":
        return {"kind": kind, "matrix": "stencil7", "N": _odd(rng, 24, 127), "fmt": rng.choice(["csr", "ell"]),
                "dtype": rng.choice(["f32", "f16"])}
    return {"kind": "batch", "count": rng.randint(4, 32), "mix": rng.randint(2, 1 << 20)}


# ------------------------------------------------------------------ matrices
def _grid(matrix, N):
    """(dimensions, offsets, values by offset; None: random values)."""
    if matrix == "poisson2d":
        off = [(0, -1), (-1, 0), (0, 0), (1, 0), (0, 1)]
        return 2, off, [4.0 if o == (0, 0) else -1.0 for o in off]
    if matrix == "stencil27":
        return 3, [(i, j, k) for k in (-1, 0, 1) for j in (-1, 0, 1) for i in (-1, 0, 1)], None
    off = [(0, 0, -1), (0, -1, 0), (-1, 0, 0), (0, 0, 0), (1, 0, 0), (0, 1, 0), (0, 0, 1)]
    if matrix == "stencil7":
        return 3, off, [6.0 if o == (0, 0, 0) else -1.0 for o in off]
    if matrix == "aniso7":
        return 3, off, [4.02 if o == (0, 0, 0) else (-0.01 if o[2] else -1.0) for o in off]
    return 3, off, [36.0 if o == (0, 0, 0) else (-11.0 if sum(o) < 0 else -1.0) for o in off]  # convdiff7


def _csr(matrix, N, seed, values="given"):
    """rowptr, col (int32) and val (float64) on the device; values="random":
    uniform values in place of the stencil's."""
    if matrix == "spd":
        A = synth.spd_diag_dominant(N, seed=seed, device=DEV)
        return tuple(torch.from_numpy(v).to(DEV) for v in (A.rowptr, A.col, A.val))
    g = torch.Generator(device=DEV).manual_seed(seed)
    if matrix == "zipf":
        lens = torch.from_numpy(np.minimum(np.random.default_rng(seed).zipf(1.5, N), min(10_000, N))).to(DEV)
        row = torch.repeat_interleave(torch.arange(N, device=DEV), lens)
        key = row * N + torch.randint(0, N, (row.numel(),), generator=g, device=DEV)
        del row
        key = torch.unique(torch.sort(key).values)  # a column drawn twice in a row is stored once
        col = (key % N).to(torch.int32)
        lens = torch.bincount(torch.div(key, N, rounding_mode="floor"), minlength=N)
        val = torch.rand(col.numel(), generator=g, device=DEV, dtype=torch.float64) * 2 - 1
    else:
        dim, off, coeffs = _grid(matrix, N)
        n = N ** dim
        i = torch.arange(n, device=DEV)
        at = [torch.div(i, N ** a, rounding_mode="floor") % N for a in range(dim)]
        ok = torch.empty((n, len(off)), dtype=torch.bool, device=DEV)
        for k, o in enumerate(off):
            m = torch.ones(n, dtype=torch.bool, device=DEV)
            for a in range(dim):
                if o[a]:
                    m &= (at[a] + o[a] >= 0) & (at[a] + o[a] < N)
            ok[:, k] = m
        lin = torch.tensor([sum(o[a] * N ** a for a in range(dim)) for o in off], device=DEV, dtype=torch.int32)
        col = (i.to(torch.int32)[:, None] + lin[None, :])[ok]
        lens = ok.sum(1)
        if coeffs is None or values == "random":
            val = torch.rand(col.numel(), generator=g, device=DEV, dtype=torch.float64) * 2 - 1
        else:
            val = torch.tensor(coeffs, device=DEV, dtype=torch.float64).expand(n, -1)[ok]
    rowptr = torch.zeros(lens.numel() + 1, dtype=torch.int32, device=DEV)
    rowptr[1:] = torch.cumsum(lens, 0)
    return rowptr, col, val


def _uniform(n, seed):
    return torch.rand(n, generator=torch.Generator(device=DEV).manual_seed(seed * 2 + 1), device=DEV,
                      dtype=torch.float64) * 2 - 1


def _product(csr, x):
    """A x in plain torch, float64 (short rows: summed in their order)."""
    rowptr, col, val = csr
    start, lens = rowptr[:-1].long(), (rowptr[1:] - rowptr[:-1]).long()
    longest = int(lens.max())
    if longest > 64:
        row = torch.repeat_interleave(torch.arange(lens.numel(), device=DEV), lens)
        y = torch.zeros(lens.numel(), dtype=torch.float64, device=DEV)
        for a in range(0, row.numel(), 1 << 25):
            b = a + (1 << 25)
            y.index_add_(0, row[a:b], val[a:b] * x[col[a:b].long()])
        return y
    y = torch.zeros(lens.numel(), dtype=torch.float64, device=DEV)
    for k in range(longest):
        live = lens > k
        e = torch.where(live, start + k, 0)
        y += torch.where(live, val[e] * x[col[e].long()], 0.0)
    return y


def _matrix(csr, dtype="f64", fmt="csr"):
    """The library's matrix, with the row partition that a program makes once."""
    rowptr, col, val = csr
    n = rowptr.numel() - 1
    A = spx.Matrix(spx.CSR, spx.F64, n, n, col.numel(), rowptr=rowptr, colidx=col, vals=val,
                   max_row_len=int((rowptr[1:] - rowptr[:-1]).max()))
    if dtype != "f64":
        A = spx.cast_values(A, DT[dtype])
    return spx.csr_analyse(A) if fmt == "csr" else spx.convert(A, FMT[fmt])


def _mix(case):
    """(matrix, N, seed offset) of a batch's systems: half Poisson grids with N
    uniform in 32..512, half random SPD with N log-uniform in 1e3..1e6."""
    r = random.Random(case["mix"])
    out = []
    for i in range(case["count"]):
        if r.random() < 0.5:
            out.append(("poisson2d", r.randint(32, 512), i))
        else:
            out.append(("spd", int(math.exp(r.uniform(math.log(1e3), math.log(1e6)))), i))
    return out


# ------------------------------------------------------------------ the cases
SOLVE = {"cg": spx.cg_solve, "bicgstab": spx.bicgstab_solve, "gmres": spx.gmres_solve, "bicg": spx.bicg_solve,
         "pipecg": spx.pipecg_solve}


def prepare(case, seed):
    kind = case["kind"]
    if kind == "batch":
        mats, bs, xs = [], [], []
        for m, N, i in _mix(case):
            csr = _csr(m, N, seed * 1000 + i)
            mats.append(_matrix(csr))
            xs.append(_uniform(mats[-1].nrows, seed * 1000 + i))
            bs.append(_product(csr, xs[-1]))
        return {"case": case, "mats": mats, "bs": bs}
    csr = _csr(case["matrix"], case["N"], seed, "random" if kind in ("convert", "transpose") else "given")
    n = csr[0].numel() - 1
    if kind == "spmv":
        A = _matrix(csr, case["dtype"], case["fmt"])
        x = _uniform(n, seed).to(A.vec_dtype)
        return {"case": case, "A": A, "x": x, "y": _uniform(n, seed + 1).to(A.vec_dtype)}
    if kind in ("convert", "transpose"):
        return {"case": case, "A": _matrix(csr, case["dtype"])}
    b = _product(csr, _uniform(n, seed))
    A = _matrix(csr, "f64", case["fmt"])
    if kind == "solve":
        return {"case": case, "A": A, "b": b}
    return {"case": case, "A": A, "low": spx.cast_values(A, DT[case["dtype"]]), "b": b}


def _arrays(M):
    """The arrays that a converted matrix holds."""
    out = {}
    for k in ("rowptr", "rowidx", "colidx", "vals", "slice_sets", "ell_col", "ell_val"):
        t = getattr(M, k)
        if t is not None and t.numel():
            out[k] = t
    return out


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "spmv":
        return spx.spmv(state["A"], state["x"], state["y"], beta=case["beta"])
    if kind == "convert":
        M = spx.convert(state["A"], FMT[case["fmt"]])
        return {"to": _arrays(M), "back": _arrays(spx.convert(M, spx.CSR))}
    if kind == "transpose":
        return _arrays(spx.csr_transpose(state["A"]))
    if kind == "solve":
        x, _ = SOLVE[case["solver"]](state["A"], state["b"], tol=1e-10, maxit=5000, precond=case["precond"])
        return x
    if kind == "ir":
        x, _ = spx.ir_solve(state["A"], state["low"], state["b"], tol=1e-10, inner_tol=1e-6)
        return x
    xs, _ = spx.cg_batch(state["mats"], state["bs"], tol=1e-8)
    return xs


def exact(case, seed):
    """The products in float64 of the stored values, the moved values, and the
    solutions that the right-hand sides were made from."""
    kind = case["kind"]
    if kind == "batch":
        return [_uniform(N * N if m == "poisson2d" else N, seed * 1000 + i) for m, N, i in _mix(case)]
    if kind in ("solve", "ir"):
        dim = 1 if case["matrix"] == "spd" else _grid(case["matrix"], case["N"])[0]
        return _uniform(case["N"] ** dim, seed)
    rowptr, col, val = _csr(case["matrix"], case["N"], seed, "given" if kind == "spmv" else "random")
    stored = {"f64": torch.float64, "f32": torch.float32, "f16": torch.float16}[case["dtype"]]
    vec = torch.float64 if case["dtype"] == "f64" else torch.float32
    val = val.to(stored).double()
    n = rowptr.numel() - 1
    if kind == "spmv":
        y = _product((rowptr, col, val), _uniform(n, seed).to(vec).double())
        return y + case["beta"] * _uniform(n, seed + 1).to(vec).double() if case["beta"] else y
    if kind == "convert":
        return {"to": None, "back": {"rowptr": None, "colidx": None, "vals": val}}
    return {"rowptr": None, "colidx": None, "vals": val[torch.sort(col, stable=True).indices]}


# ------------------------------------------------------------------ work
def _shape(matrix, N):
    """Rows and (for the random matrices: expected) entries."""
    if matrix == "zipf":
        return N, 151.0 * N if N >= 100_000 else 140.0 * N
    if matrix == "spd":
        return N, 16.5 * N
    dim, off, _ = _grid(matrix, N)
    return N ** dim, float(sum(math.prod(N - abs(v) for v in o) for o in off))


def _csr_bytes(n, nnz, sv):
    return nnz * (sv + 4) + 4 * (n + 1)


def _fmt_bytes(fmt, matrix, n, nnz, sv):
    if fmt == "csr":
        return _csr_bytes(n, nnz, sv)
    if fmt == "coo" or (fmt == "hyb" and matrix == "zipf"):
        return nnz * (sv + 8)
    return nnz * (sv + 4)  # slot arrays, without the padding


# iterations to the tolerances above: about this many per grid edge (spd: in all)
_ITERS = {("cg", "poisson2d"): 3.2, ("cg", "aniso7"): 4.4, ("cg", "stencil7"): 3.15, ("cg", "spd"): 37,
          ("bicgstab", "convdiff7"): 2.6, ("gmres", "convdiff7"): 4.9, ("bicg", "convdiff7"): 4.8}


def _solve_work(solver, matrix, N, precond, sv=8, sx=8, iters=None):
    n, nnz = _shape(matrix, N)
    base = "cg" if solver == "pipecg" else solver
    it = iters if iters is not None else _ITERS[base, matrix] * (1 if matrix == "spd" else N)
    products = 2 if solver in ("bicgstab", "bicg") else 1
    # the vectors that one step reads and writes (GMRES(30): the basis of 15
    # vectors on average, read twice)
    vectors = {"cg": 8 + 2 * precond, "pipecg": 8 + 2 * precond, "bicgstab": 15 + 2 * precond, "bicg": 14 + 2 * precond,
               "gmres": 2 * 15.5 + 4 + precond}[solver]
    step = products * _csr_bytes(n, nnz, sv) + (2 * products + vectors) * n * sx
    flops = products * 2 * nnz + 2 * vectors * n
    if n <= 4096:  # held on chip for the whole solve
        return {"bytes": _csr_bytes(n, nnz, sv) + 2 * n * sx, "flops": it * flops}
    return {"bytes": it * step, "flops": it * flops}


def work(case):
    kind = case["kind"]
    if kind == "batch":
        each = [_solve_work("cg", m, N, 0, iters=1.85 * N if m == "poisson2d" else 29) for m, N, _ in _mix(case)]
        return {k: sum(w[k] for w in each) for k in ("bytes", "flops")}
    if kind == "solve":
        return _solve_work(case["solver"], case["matrix"], case["N"], case["precond"])
    if kind == "ir":
        return _solve_work("cg", case["matrix"], case["N"], 0, SIZE[case["dtype"]], 4, iters=3.3 * case["N"])
    n, nnz = _shape(case["matrix"], case["N"])
    sv = SIZE[case["dtype"]]
    if kind == "spmv":
        sx = 8 if case["dtype"] == "f64" else 4
        return {"bytes": _fmt_bytes(case["fmt"], case["matrix"], n, nnz, sv) + n * sx * (3 if case["beta"] else 2),
                "flops": 2 * nnz}
    if kind == "convert":
        return {"bytes": 2 * (_csr_bytes(n, nnz, sv) + _fmt_bytes(case["fmt"], case["matrix"], n, nnz, sv)), "flops": 0}
    return {"bytes": 2 * _csr_bytes(n, nnz, sv), "flops": 0}
