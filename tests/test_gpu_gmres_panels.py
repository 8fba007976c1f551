"""GMRES at the edges of its basis layout: sizes around one panel of 256 rows,
restart lengths around the register groups of the pass kernels, and systems
scaled far from one (the basis is stored unscaled), against the CPU oracle."""
import numpy as np
import pytest

import oracle as O
from paper_2006_14290_amd import synth as S

from gpu_util import dev, host

pytestmark = pytest.mark.gpu

spx = pytest.importorskip("paper_2006_14290_amd.spx")


def tridiagonal(n, scale=1.0):
    d = np.zeros((n, 3))
    d[:, 0], d[:, 1], d[:, 2] = -2.0, 4.0 + np.arange(n) % 3, -1.0
    cols = np.arange(n)[:, None] + np.array([-1, 0, 1])
    ok = (cols >= 0) & (cols < n)
    rowptr = np.concatenate([[0], np.cumsum(ok.sum(1))])
    return S.CSR(n, rowptr.astype(np.int32), cols[ok].astype(np.int32), scale * d[ok])


def solve_both(A, restart, precond):
    b = O.csr_spmv(A, S.uniform_vector(A.n, seed=3, purpose="xstar"))
    x, info = spx.gmres_solve(spx.csr_from_host(A), dev(b), tol=1e-10, precond=precond, restart=restart, maxit=3000)
    xo, io = O.gmres(A, b, tol=1e-10, precond=precond, restart=restart, maxit=3000)
    assert info["status"] == spx.OK and io["status"] == O.OK, (info, io)
    assert abs(info["iters"] - io["iters"]) <= 0.1 * io["iters"] + 5, (info["iters"], io["iters"])
    r = b - O.csr_spmv(A, host(x))
    assert np.linalg.norm(r) <= 1.01e-10 * np.linalg.norm(b)


@pytest.mark.parametrize("restart", [1, 4, 5, 16, 33, 62])
@pytest.mark.parametrize("n", [1, 5, 255, 256, 257, 1000, 70001])
def test_panel_and_group_edges(n, restart):
    print(f"case n={n} restart={restart}", flush=True)
    A = tridiagonal(n)
    for precond in (0, 1):
        solve_both(A, restart, precond)


@pytest.mark.parametrize("scale", [1e-100, 1e100])
def test_scaled_systems(scale):
    print(f"case scale={scale}", flush=True)
    solve_both(tridiagonal(1000, scale), 30, 0)
