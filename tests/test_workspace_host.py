"""The solvers' workspace depends on a matrix's sizes only: not on its
row-length hint or on where its arrays lie, which decide the kernel. A
workspace queried before the hint is set, or for a copy at other addresses, is
accepted by the solve (which carves it by the same function). No GPU."""
import ctypes

import pytest

from test_abi import lib  # noqa: F401  (fixture)

CSR, ELL = 0, 2


class Desc(ctypes.Structure):
    _fields_ = [("fmt", ctypes.c_int32), ("val_type", ctypes.c_int32), ("nrows", ctypes.c_int32),
                ("ncols", ctypes.c_int32), ("nnz", ctypes.c_int64), ("rowptr", ctypes.c_void_p),
                ("rowidx", ctypes.c_void_p), ("colidx", ctypes.c_void_p), ("vals", ctypes.c_void_p),
                ("coo_nnz", ctypes.c_int64), ("ell_width", ctypes.c_int32), ("max_row_len", ctypes.c_int32),
                ("ell_ld", ctypes.c_int64), ("ell_col", ctypes.c_void_p), ("ell_val", ctypes.c_void_p),
                ("csr_part", ctypes.c_void_p), ("slice_size", ctypes.c_int32), ("stride_factor", ctypes.c_int32),
                ("slice_sets", ctypes.c_void_p), ("slice_cols", ctypes.c_int64),
                ("csr_cb", ctypes.c_void_p), ("csr_cb_tiles", ctypes.c_int32), ("csr_cb_live", ctypes.c_int32)]


class Opts(ctypes.Structure):
    _fields_ = [("tol", ctypes.c_double), ("maxit", ctypes.c_int32), ("restart", ctypes.c_int32),
                ("precond", ctypes.c_int32), ("x0_zero", ctypes.c_int32), ("check_every", ctypes.c_int32),
                ("reserved", ctypes.c_int32)]


def workspace(lib, solver, precond=0, restart=1, **kw):
    d = Desc(val_type=0, **kw)
    d.ncols = d.nrows
    out = ctypes.c_size_t(0)
    lib.spx_solve_workspace.argtypes = [ctypes.c_int32, ctypes.POINTER(Desc), ctypes.POINTER(Opts),
                                        ctypes.POINTER(ctypes.c_size_t)]
    assert lib.spx_solve_workspace(solver, d, Opts(tol=1e-8, maxit=10, restart=restart, precond=precond), out) == 0
    return out.value


@pytest.mark.parametrize("solver", range(5))
@pytest.mark.parametrize("n,per", [(1, 1), (100, 5), (1639, 5), (4097, 5), (20_000, 16), (32_768, 64), (32_769, 60),
                                   (50_000, 27), (300_000, 7), (300_000, 120), (3_000_000, 5)])
def test_csr_hint_and_addresses(lib, n, per, solver):  # noqa: F811
    got = {workspace(lib, solver, fmt=CSR, nrows=n, nnz=n * per, rowptr=0x10000, colidx=c, vals=v, max_row_len=hint)
           for hint in (0, per, per + 3, 2 * per, 10 * per)
           for c, v in ((0x20000, 0x30000), (0x20004, 0x30000), (0x20000, 0x30008))}
    assert len(got) == 1, sorted(got)


@pytest.mark.parametrize("solver", [0, 1, 2, 4])
@pytest.mark.parametrize("n", [1, 257, 300_000, 3_000_000])
def test_ell_addresses(lib, n, solver):  # noqa: F811
    got = {workspace(lib, solver, fmt=ELL, nrows=n, nnz=n * 7, ell_width=7, ell_ld=ld, ell_col=c, ell_val=v)
           for ld in (n, n + 1) for c, v in ((0x20000, 0x30000), (0x20004, 0x30000), (0x20000, 0x30008))}
    assert len(got) == 1, sorted(got)


def test_cg_vectors(lib):  # noqa: F811
    """Jacobi CG keeps the diagonal and its inverse besides plain CG's
    vectors, block Jacobi z and the inverse blocks."""
    n = 1 << 16  # a vector is a whole number of 256-byte pieces

    def cg(precond):
        return workspace(lib, 0, precond, fmt=CSR, nrows=n, nnz=7 * n, rowptr=0x10000, colidx=0x20000, vals=0x30000)

    assert cg(1) - cg(0) == 2 * 8 * n
    assert cg(2) - cg(0) == 3 * 8 * n
