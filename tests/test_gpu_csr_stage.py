"""GPU parity of the staged-rows CSR product (rows of similar, known length)
at the edges of its classes: full and ragged rows, partial last blocks, entry
counts that end inside a 16-byte vector, wrong hints, infinities, and the
fused dot products, against the CPU oracle."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2006_14290_amd import synth as S

from gpu_util import assert_spmv_f64, assert_spmv_low, dev, host

pytestmark = pytest.mark.gpu

spx = pytest.importorskip("paper_2006_14290_amd.spx")

N = 66001  # above the row-per-subwarp kernel's range; the last block is partial


def banded(n, lo, hi, seed, extra=0):
    """Rows of lo..hi entries near the diagonal; `extra` more rows of one
    entry move the entry count off a multiple of 8."""
    r = np.random.default_rng(seed)
    lens = r.integers(lo, hi + 1, n)
    lens[:extra] = lo - 1 if lo > 1 else lo
    rowptr = np.concatenate([[0], np.cumsum(lens)])
    step = r.integers(1, 4, rowptr[-1])
    cum = np.concatenate([[0], np.cumsum(step)])
    base = np.clip(np.arange(n) - hi, 0, n - 3 * hi - 4)
    col = np.repeat(base - cum[rowptr[:-1]], lens) + cum[:-1]
    return S.CSR(n, rowptr.astype(np.int32), col.astype(np.int32), r.uniform(-1, 1, rowptr[-1]))


def rounded(v, dtype):
    return np.asarray(v, {"f64": np.float64, "f32": np.float32, "f16": np.float16}[dtype]).astype(np.float64)


def check(A, Ad, dtype, alpha=1.0, beta=0.0):
    vec = "f64" if dtype == "f64" else "f32"
    x, y0 = rounded(S.uniform_vector(A.n, seed=1), vec), rounded(S.uniform_vector(A.n, seed=2), vec)
    yref, absax = O.csr_spmv_dot2(S.CSR(A.n, A.rowptr, A.col, rounded(A.val, dtype)), x, y0, alpha=alpha, beta=beta)
    y = host(spx.spmv(Ad, dev(x, Ad.vec_dtype), dev(y0, Ad.vec_dtype), alpha=alpha, beta=beta))
    if dtype == "f64":
        assert_spmv_f64(y, yref, abs(alpha) * absax, beta_y=beta * y0)
    else:
        assert_spmv_low(y, yref, abs(alpha) * absax, np.diff(A.rowptr), beta_y=beta * y0)


@pytest.mark.parametrize("dtype", ["f64", "f32", "f16"])
@pytest.mark.parametrize("lo,hi", [(3, 8), (8, 8), (9, 16), (16, 16), (17, 32), (27, 27), (33, 64), (70, 128)])
def test_row_length_classes(lo, hi, dtype):
    print(f"case {lo}..{hi} {dtype}", flush=True)
    for extra in (0, 3):
        A = banded(N, lo, hi, seed=lo * 100 + hi, extra=extra)
        Ad = spx.csr_from_host(A, spx.DTYPE_NAMES[dtype])
        check(A, Ad, dtype)
    check(A, Ad, dtype, alpha=-2.5, beta=0.75)


@pytest.mark.parametrize("dtype", ["f64", "f32", "f16"])
def test_wrong_hint_and_unaligned_arrays(dtype):
    """A hint below the longest row, and arrays that do not start on a 16-byte
    boundary (another kernel takes those): same result."""
    A = banded(N, 3, 8, seed=5)
    lens = np.diff(A.rowptr).astype(np.int64)
    for r in (0, 4000, N - 1):  # rows far longer than the hint says
        lens[r] = 3000
    rowptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    col = np.concatenate([np.arange(l) if l == 3000 else A.col[A.rowptr[i]:A.rowptr[i + 1]]
                          for i, l in enumerate(lens)]).astype(np.int32)
    B = S.CSR(N, rowptr, col, np.random.default_rng(6).uniform(-1, 1, rowptr[-1]))
    Bd = spx.csr_from_host(B, spx.DTYPE_NAMES[dtype])
    Bd.max_row_len = 8
    check(B, Bd, dtype)
    Ad = spx.csr_from_host(A, spx.DTYPE_NAMES[dtype])
    for k in ("colidx", "vals"):
        t = getattr(Ad, k)
        u = torch.empty(t.numel() + 1, dtype=t.dtype, device=t.device)[1:]
        u.copy_(t)
        setattr(Ad, k, u)
    check(A, Ad, dtype)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_infinities_stay_in_their_rows(dtype):
    """x[0] = inf and NaN in y (beta = 0) reach only the rows that hold column 0."""
    A = banded(N, 3, 8, seed=7)
    Ad = spx.csr_from_host(A, spx.DTYPE_NAMES[dtype])
    x = rounded(S.uniform_vector(A.n, seed=1), dtype)
    x[0] = np.inf
    y = host(spx.spmv(Ad, dev(x, Ad.vec_dtype), torch.full((A.n,), float("nan"), dtype=Ad.vec_dtype, device="cuda")))
    has0 = np.zeros(A.n, bool)
    has0[np.repeat(np.arange(A.n), np.diff(A.rowptr))[A.col == 0]] = True
    assert has0.any() and np.all(np.isinf(y[has0])) and np.all(np.isfinite(y[~has0]))


def test_fused_dots_and_reproducibility():
    """CG and BiCGSTAB above the small sizes use the epilogue sums: iteration
    counts and residuals follow the oracle, and a repeated solve is bitwise
    the same."""
    A = S.poisson2d(260)
    Ad = spx.csr_from_host(A)
    b = O.csr_spmv(A, S.uniform_vector(A.n, seed=1, purpose="xstar"))
    bd = dev(b)
    for solve, oracle in ((spx.cg_solve, O.cg), (spx.bicgstab_solve, O.bicgstab)):
        x, info = solve(Ad, bd, tol=1e-8)
        _, ref = oracle(A, b, tol=1e-8, maxit=10000)
        assert info["status"] == 0 and info["iters"] <= 1.1 * ref["iters"] + 5
        r = b - O.csr_spmv(A, host(x))
        assert np.linalg.norm(r) <= 1.01e-8 * np.linalg.norm(b)
        x2, _ = solve(Ad, bd, tol=1e-8)
        np.testing.assert_array_equal(host(x).view(np.uint64), host(x2).view(np.uint64))
