"""The ELL product above 2^18 rows, where the gathers' order depends on the
rows: ragged rows (less than half of the slots stored), scattered and banded
full rows and both in one matrix; odd and even row counts and leading
dimensions, rows of one entry, binary16 rows below and from 8 entries;
products and the solvers' fused sums, against the CPU oracle."""
import numpy as np
import pytest

import oracle as O
from paper_2006_14290_amd import synth as S

from gpu_util import assert_spmv_f64, assert_spmv_low, dev, host

pytestmark = pytest.mark.gpu

spx = pytest.importorskip("paper_2006_14290_amd.spx")

LARGE = 1 << 18  # rows up to which every row's gathers go out together


def rows(kind, n, K, seed=1):
    """n x n: K entries per row (ragged: 0 to K, most rows short)."""
    r = np.random.default_rng(seed)
    band = np.minimum(np.arange(n)[:, None] // 2, n - K) + np.arange(K)
    # one random column out of each K-th of the range: ascending and distinct
    wide = np.arange(K) * (n // K) + r.integers(0, n // K, (n, K))
    col = band if kind == "banded" else wide
    if kind == "mixed":
        col = np.where((np.arange(n) // 1000 % 2 == 0)[:, None], band, wide)
    keep = np.ones((n, K), bool)
    if kind == "ragged":
        lens = np.minimum(r.geometric(0.3, n) - 1, K)
        lens[n // 2] = K
        keep = np.arange(K) < lens[:, None]
    rowptr = np.concatenate([[0], np.cumsum(keep.sum(1))])
    return S.CSR(n, rowptr.astype(np.int32), col[keep].astype(np.int32), r.uniform(-1, 1, int(rowptr[-1])))


@pytest.mark.parametrize("dtype", ["f64", "f32", "f16"])
@pytest.mark.parametrize("kind,n,K", [("ragged", LARGE + 1, 13), ("ragged", LARGE + 514, 8), ("wide", LARGE, 9),
                                      ("wide", LARGE + 1, 9), ("wide", LARGE + 2, 8), ("banded", LARGE + 127, 11),
                                      ("banded", LARGE + 640, 7), ("mixed", LARGE + 3, 12), ("wide", LARGE + 2, 1),
                                      ("wide", LARGE + 5, 5)])
def test_products(kind, n, K, dtype):
    print(f"case {kind} n={n} K={K} {dtype}", flush=True)
    A = rows(kind, n, K)
    vec = np.float64 if dtype == "f64" else np.float32
    stored = A.val.astype({"f64": np.float64, "f32": np.float32, "f16": np.float16}[dtype]).astype(np.float64)
    x = S.uniform_vector(n, seed=1).astype(vec).astype(np.float64)
    y0 = S.uniform_vector(n, seed=2).astype(vec).astype(np.float64)
    Ad = spx.csr_from_host(A, spx.DTYPE_NAMES[dtype])
    lens = np.diff(A.rowptr)
    for fmt, ld in ((spx.ELL, n + n % 2), (spx.ELL, n + 1 - n % 2), (spx.HYB, n + n % 2)):
        M = spx.convert(Ad, fmt, ell_width=K if fmt == spx.ELL else max(1, K - 1), ell_ld=ld)
        for alpha, beta in ((1.0, 0.0), (-1.5, 0.5)):
            yref, absax = O.csr_spmv_dot2(S.CSR(n, A.rowptr, A.col, stored), x, y0, alpha=alpha, beta=beta)
            y = host(spx.spmv(M, dev(x, M.vec_dtype), dev(y0, M.vec_dtype), alpha=alpha, beta=beta))
            if dtype == "f64":
                assert_spmv_f64(y, yref, abs(alpha) * absax, beta_y=beta * y0)
            else:
                assert_spmv_low(y, yref, abs(alpha) * absax, lens, beta_y=beta * y0)


@pytest.mark.parametrize("kind", ["spd", "grid"])
def test_solvers_sums(kind):
    """CG and refinement through the fused product and sums of the ELL kernel."""
    print(f"case {kind}", flush=True)
    A = S.spd_diag_dominant(LARGE + 1000, seed=3, device="cuda") if kind == "spd" else S.poisson2d(513)
    b, _ = O.csr_spmv_dot2(A, S.uniform_vector(A.n, seed=4))
    M = spx.convert(spx.csr_from_host(A), spx.ELL)
    x, info = spx.cg_solve(M, dev(b), tol=1e-9, maxit=4000)
    assert info["status"] == spx.OK, info
    assert np.linalg.norm(b - O.csr_spmv(A, host(x))) <= 1.01e-9 * np.linalg.norm(b)
    for low in (spx.F32, spx.F16):
        x, info = spx.ir_solve(M, spx.cast_values(M, low), dev(b), tol=1e-9, inner_tol=1e-4)
        assert info["status"] == spx.OK, info
        assert np.linalg.norm(b - O.csr_spmv(A, host(x))) <= 1.01e-9 * np.linalg.norm(b)
