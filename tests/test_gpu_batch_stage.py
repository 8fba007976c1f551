"""Wide batched solves over the product's two forms (tiles, staged rows): row
lengths at the edges of the staged classes, row counts that end inside a
wavefront's block, one long row, arrays that 16-byte copies cannot read, few
entries, and systems that finish far apart; each against its true residual in
float64, and bit for bit against the system solved alone."""
import numpy as np
import pytest
import torch

from paper_2006_14290_amd import synth as S

from gpu_util import dev, host

pytestmark = pytest.mark.gpu

spx = pytest.importorskip("paper_2006_14290_amd.spx")

TOL = 1e-10


def spd_band(n, half, seed, long_row=0):
    """Symmetric, diagonally dominant: a diagonal and `half` off-diagonals on
    each side (2 * half + 1 entries in full rows); long_row couples the first
    row to that many others."""
    r = np.random.default_rng(seed)
    i = np.arange(n)
    rows, cols = [], []
    for d in range(1, half + 1):
        rows.append(i[d:]), cols.append(i[:-d])
    if long_row:
        far = half + 1 + np.arange(long_row)
        rows.append(far), cols.append(np.zeros(long_row, int))
    rows, cols = np.concatenate(rows), np.concatenate(cols)
    v = -r.uniform(0.5, 1.0, rows.size)
    diag = np.full(n, 0.05)
    np.add.at(diag, rows, -v)
    np.add.at(diag, cols, -v)
    R, C = np.concatenate([rows, cols, i]), np.concatenate([cols, rows, i])
    V = np.concatenate([v, v, diag])
    o = np.lexsort((C, R))
    rowptr = np.concatenate([[0], np.cumsum(np.bincount(R, minlength=n))])
    return S.CSR(n, rowptr.astype(np.int32), C[o].astype(np.int32), V[o])


def device(A, shift=0):
    """shift: entries by which the arrays start off a 16-byte boundary."""
    if not shift:
        return spx.csr_from_host(A)
    col = torch.cat([torch.zeros(shift, dtype=torch.int32), torch.from_numpy(A.col)]).cuda()[shift:]
    val = torch.cat([torch.zeros(shift, dtype=torch.float64), torch.from_numpy(A.val)]).cuda()[shift:]
    return spx.Matrix(spx.CSR, spx.F64, A.n, A.n, A.col.size, rowptr=torch.from_numpy(A.rowptr).cuda(), colidx=col,
                      vals=val)


SYSTEMS = {
    "rows of 3, few entries": (spd_band(2000, 1, 1), 0),  # below kStageMinNnz
    "rows of 3": (spd_band(5000, 1, 2), 0),               # too short for the class of 8
    "rows of 5": (spd_band(30001, 2, 3), 0),
    "rows of 7, odd block": (spd_band(4096 + 65, 3, 4), 0),
    "rows of 7, odd arrays": (spd_band(9000, 3, 5), 1),
    "rows of 9": (spd_band(20479, 4, 6), 0),
    "rows of 17": (spd_band(6000, 8, 7), 0),
    "rows of 31": (spd_band(5555, 15, 8), 0),
    "rows of 63": (spd_band(5000, 31, 9), 0),
    "rows of 127": (spd_band(4100, 63, 10), 0),
    "rows of 131": (spd_band(4200, 65, 11), 0),            # past every class
    "one long row": (spd_band(12000, 2, 12, long_row=3000), 0),
    "grid 150^2": (S.poisson2d(150), 0),
}


def check(A, b, x, info):
    assert info["status"] == spx.OK, info
    y = np.zeros(A.n)
    np.add.at(y, np.repeat(np.arange(A.n), np.diff(A.rowptr)), A.val * x[A.col])
    # the solver's own true residual is at most TOL; the two evaluations of
    # A x differ by a few eps * |A| |x| per row
    ax = np.zeros(A.n)
    np.add.at(ax, np.repeat(np.arange(A.n), np.diff(A.rowptr)), np.abs(A.val * x[A.col]))
    slack = 2.0 ** -52 * np.diff(A.rowptr).max() * np.linalg.norm(ax)
    assert np.linalg.norm(b - y) <= TOL * np.linalg.norm(b) + slack


def test_wide_forms_solve_and_do_not_depend_on_the_mix():
    mats = {k: device(A, sh) for k, (A, sh) in SYSTEMS.items()}
    bs = {k: S.uniform_vector(A.n, seed=j) for j, (k, (A, _)) in enumerate(SYSTEMS.items())}
    print("case mix", flush=True)
    xs, infos = spx.cg_batch([mats[k] for k in SYSTEMS], [dev(bs[k]) for k in SYSTEMS], tol=TOL,
                             path=spx.BATCH_WIDE)
    for k, x, info in zip(SYSTEMS, xs, infos):
        print(f"case {k}", flush=True)
        check(SYSTEMS[k][0], bs[k], host(x), info)
        xa, ia = spx.cg_batch([mats[k]], [dev(bs[k])], tol=TOL, path=spx.BATCH_WIDE)
        assert ia[0]["iters"] == info["iters"]
        assert torch.equal(xa[0], x), k


def test_staged_bicgstab_through_the_server():
    A, _ = SYSTEMS["rows of 7, odd block"]
    B = S.CSR(A.n, A.rowptr, A.col, A.val * np.where(A.col > np.repeat(np.arange(A.n), np.diff(A.rowptr)), 0.7, 1.0))
    b = S.uniform_vector(A.n, seed=40)
    print("case bicgstab", flush=True)
    srv = spx.Server(max_slots=4, hbm_budget_bytes=1 << 28)
    try:
        for M, solver in ((B, spx.SOLVER_BICGSTAB), (A, spx.SOLVER_CG)):
            x, info = srv.wait(srv.submit(M, b, tol=TOL, solver=solver), 60.0)
            check(M, b, np.asarray(x), info)
    finally:
        srv.close()
