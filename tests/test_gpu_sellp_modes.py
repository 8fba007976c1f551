"""SELL-P products in 64-row slices where a wavefront looks for scattered
rows: 2^16 to 2^17 rows, and float64 with x above 4 MB; scattered, banded and
mixed rows, lengths around the eight slot columns taken at once, a last slice
that is not full, against the CPU oracle."""
import numpy as np
import pytest

import oracle as O
from paper_2006_14290_amd import synth as S

from gpu_util import assert_spmv_f64, assert_spmv_low, dev, host
from test_gpu_ell_modes import rows

pytestmark = pytest.mark.gpu

spx = pytest.importorskip("paper_2006_14290_amd.spx")


@pytest.mark.parametrize("dtype", ["f64", "f32", "f16"])
@pytest.mark.parametrize("kind,n,K", [("wide", (1 << 16) + 1, 8), ("wide", 70_000, 9), ("wide", 1 << 17, 17),
                                      ("banded", 100_001, 16), ("mixed", 130_003, 31), ("ragged", 90_000, 24),
                                      ("wide", 524_289, 9), ("banded", 530_000, 8), ("mixed", 600_001, 10)])
def test_products(kind, n, K, dtype):
    print(f"case {kind} n={n} K={K} {dtype}", flush=True)
    A = rows(kind, n, K)
    vec = np.float64 if dtype == "f64" else np.float32
    stored = A.val.astype({"f64": np.float64, "f32": np.float32, "f16": np.float16}[dtype]).astype(np.float64)
    x = S.uniform_vector(n, seed=1).astype(vec).astype(np.float64)
    y0 = S.uniform_vector(n, seed=2).astype(vec).astype(np.float64)
    M = spx.convert(spx.csr_from_host(A, spx.DTYPE_NAMES[dtype]), spx.SELLP)
    for alpha, beta in ((1.0, 0.0), (-1.5, 0.5)):
        yref, absax = O.csr_spmv_dot2(S.CSR(n, A.rowptr, A.col, stored), x, y0, alpha=alpha, beta=beta)
        y = host(spx.spmv(M, dev(x, M.vec_dtype), dev(y0, M.vec_dtype), alpha=alpha, beta=beta))
        if dtype == "f64":
            assert_spmv_f64(y, yref, abs(alpha) * absax, beta_y=beta * y0)
        else:
            assert_spmv_low(y, yref, abs(alpha) * absax, np.diff(A.rowptr), beta_y=beta * y0)


@pytest.mark.parametrize("n", [100_000, 530_000])
def test_solvers_sums(n):
    print(f"case n={n}", flush=True)
    A = S.spd_diag_dominant(n, seed=3, device="cuda")
    b, _ = O.csr_spmv_dot2(A, S.uniform_vector(n, seed=4))
    x, info = spx.cg_solve(spx.convert(spx.csr_from_host(A), spx.SELLP), dev(b), tol=1e-9, maxit=4000)
    assert info["status"] == spx.OK, info
    assert np.linalg.norm(b - O.csr_spmv(A, host(x))) <= 1.01e-9 * np.linalg.norm(b)
