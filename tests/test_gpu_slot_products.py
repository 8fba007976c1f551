"""GPU parity of the ELL, SELL-P and COO products where the slot columns or
entries in flight end: widths around the multiples of a block of slots, ragged
and empty rows, odd and even row counts and leading dimensions, slice sizes
with one and several lane groups, chunks that end early, infinities at column
0 (which padding must not read into a sum), against the CPU oracle."""
import numpy as np
import pytest

import oracle as O
from paper_2006_14290_amd import synth as S

from gpu_util import assert_spmv_f64, assert_spmv_low, dev, host

pytestmark = pytest.mark.gpu

spx = pytest.importorskip("paper_2006_14290_amd.spx")


def ragged(n, width, seed):
    """Rows of 0..width entries, at least one of width."""
    r = np.random.default_rng(seed)
    lens = r.integers(0, width + 1, n)
    lens[r.integers(0, n)] = width
    rowptr = np.concatenate([[0], np.cumsum(lens)])
    col = np.concatenate([np.sort(r.choice(n, k, replace=False)) for k in lens])
    return S.CSR(n, rowptr.astype(np.int32), col.astype(np.int32), r.uniform(-1, 1, rowptr[-1]))


def rounded(v, dtype):
    return np.asarray(v, {"f64": np.float64, "f32": np.float32, "f16": np.float16}[dtype]).astype(np.float64)


def check(A, Ad, dtype, alpha, beta):
    vec = "f64" if dtype == "f64" else "f32"
    x, y0 = rounded(S.uniform_vector(A.n, seed=1), vec), rounded(S.uniform_vector(A.n, seed=2), vec)
    yref, absax = O.csr_spmv_dot2(S.CSR(A.n, A.rowptr, A.col, rounded(A.val, dtype)), x, y0, alpha=alpha, beta=beta)
    y = host(spx.spmv(Ad, dev(x, Ad.vec_dtype), dev(y0, Ad.vec_dtype), alpha=alpha, beta=beta))
    if dtype == "f64":
        assert_spmv_f64(y, yref, abs(alpha) * absax, beta_y=beta * y0)
    else:
        assert_spmv_low(y, yref, abs(alpha) * absax, np.diff(A.rowptr), beta_y=beta * y0)


@pytest.mark.parametrize("dtype", ["f64", "f32", "f16"])
@pytest.mark.parametrize("width", [1, 3, 4, 5, 7, 8, 9, 15, 16, 17, 33])
def test_widths(width, dtype):
    print(f"case width {width} {dtype}", flush=True)
    for n in (130, 1027):
        A = ragged(n, width, seed=width * 10 + n)
        Ad = spx.csr_from_host(A, spx.DTYPE_NAMES[dtype])
        check(A, spx.convert(Ad, spx.ELL), dtype, 1.0, 0.0)
        check(A, spx.convert(Ad, spx.ELL, ell_ld=n + 1 + n % 2), dtype, -1.5, 0.5)  # odd: one row per thread
        for C in (8, 64, 256):
            check(A, spx.convert(Ad, spx.SELLP, slice_size=C), dtype, -1.5, 0.5)
        check(A, spx.convert(Ad, spx.COO), dtype, 1.0, 0.0)
        check(A, spx.convert(Ad, spx.HYB, ell_width=width // 2), dtype, -1.5, 0.5)


@pytest.mark.parametrize("fmt", ["ELL", "SELLP", "COO", "HYB"])
def test_infinity_reaches_its_own_rows_only(fmt):
    print(f"case infinity {fmt}", flush=True)
    A = ragged(700, 11, seed=5)
    x = S.uniform_vector(A.n, seed=3)
    for at in (0, 350, A.n - 1):
        xi = x.copy()
        xi[at] = np.inf
        y = host(spx.spmv(spx.convert(spx.csr_from_host(A), getattr(spx, fmt)), dev(xi)))
        hit = np.zeros(A.n, bool)
        hit[np.repeat(np.arange(A.n), np.diff(A.rowptr))[A.col == at]] = True
        assert np.isinf(y[hit]).all() and np.isfinite(y[~hit]).all()


@pytest.mark.parametrize("per", [31, 33])
def test_coo_chunks_of_large_matrices(per):
    """Entry counts around the step to larger chunks (2^25 entries)."""
    n = (1 << 20) - (per == 33) * 17  # 4 MB in float32
    print(f"case coo {n} rows of {per}", flush=True)
    off = np.sort(np.random.default_rng(per).choice(4 * per, per, replace=False))
    col = np.minimum(np.arange(n)[:, None], n - 4 * per) + off
    A = S.CSR(n, (np.arange(n + 1) * per).astype(np.int32), col.reshape(-1).astype(np.int32),
              np.random.default_rng(1).uniform(-1, 1, n * per))
    for dtype in ("f64", "f32"):  # x of more and of at most 4 MB
        Ad = spx.csr_from_host(A, spx.DTYPE_NAMES[dtype])
        check(A, spx.convert(Ad, spx.COO), dtype, 1.0, 0.0)
        check(A, spx.convert(Ad, spx.HYB, ell_width=1), dtype, -1.5, 0.5)
