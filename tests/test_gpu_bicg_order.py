"""BiCG and BiCGSTAB take their sums in the tile kernel's order whether or not
the rows' length is known: the same bits with the hint as without it."""
import numpy as np
import pytest

import oracle as O
from paper_2006_14290_amd import synth as S

from gpu_util import dev, host

pytestmark = pytest.mark.gpu

spx = pytest.importorskip("paper_2006_14290_amd.spx")


@pytest.mark.parametrize("solver", ["bicg_solve", "bicgstab_solve"])
@pytest.mark.parametrize("precond", [0, 1])
def test_row_length_hint(solver, precond):
    print(f"case {solver} precond={precond}", flush=True)
    A = S.convdiff3d_upwind(40)
    b = O.csr_spmv(A, S.uniform_vector(A.n, seed=2))
    Ad = spx.csr_from_host(A)
    assert Ad.max_row_len == 7 and A.n > 32768
    plain = spx.Matrix(spx.CSR, spx.F64, A.n, A.n, Ad.nnz, rowptr=Ad.rowptr, colidx=Ad.colidx, vals=Ad.vals)
    x, info = getattr(spx, solver)(Ad, dev(b), tol=1e-10, precond=precond)
    y, _ = getattr(spx, solver)(plain, dev(b), tol=1e-10, precond=precond)
    assert info["status"] == spx.OK
    np.testing.assert_array_equal(host(x).view(np.uint64), host(y).view(np.uint64))
