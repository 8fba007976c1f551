"""BiCG above 65,536 rows and BiCGSTAB above 2^18 take their sums in the tile
kernel's order whether or not the rows' length is known: the same bits with
the hint as without it. BiCG's short known rows take the row-per-subwarp kernel
from 32,769 to 65,536 rows, several steps to a work-group: against the oracle."""
import numpy as np
import pytest

import oracle as O
from paper_2006_14290_amd import synth as S

from gpu_util import dev, host

pytestmark = pytest.mark.gpu

spx = pytest.importorskip("paper_2006_14290_amd.spx")


@pytest.mark.parametrize("solver,N", [("bicg_solve", 41), ("bicgstab_solve", 65)])
@pytest.mark.parametrize("precond", [0, 1])
def test_row_length_hint(solver, N, precond):
    print(f"case {solver} N={N} precond={precond}", flush=True)
    A = S.convdiff3d_upwind(N)
    b = O.csr_spmv(A, S.uniform_vector(A.n, seed=2))
    Ad = spx.csr_from_host(A)
    assert Ad.max_row_len == 7
    plain = spx.Matrix(spx.CSR, spx.F64, A.n, A.n, Ad.nnz, rowptr=Ad.rowptr, colidx=Ad.colidx, vals=Ad.vals)
    x, info = getattr(spx, solver)(Ad, dev(b), tol=1e-10, precond=precond)
    y, _ = getattr(spx, solver)(plain, dev(b), tol=1e-10, precond=precond)
    assert info["status"] == spx.OK
    np.testing.assert_array_equal(host(x).view(np.uint64), host(y).view(np.uint64))


@pytest.mark.parametrize("solver", ["bicg_solve", "bicgstab_solve"])
@pytest.mark.parametrize("N", [32, 33, 40])
def test_row_kernel_steps(solver, N):
    print(f"case {solver} N={N}", flush=True)
    A = S.convdiff3d_upwind(N)
    b = O.csr_spmv(A, S.uniform_vector(A.n, seed=2))
    for precond in (0, 1):
        x, info = getattr(spx, solver)(spx.csr_from_host(A), dev(b), tol=1e-10, precond=precond)
        assert info["status"] == spx.OK
        assert np.linalg.norm(b - O.csr_spmv(A, host(x))) <= 1.01e-10 * np.linalg.norm(b)
