"""One-work-group CG (single solves and batches) at the edges of its row
ownership: row counts around wavefronts, work-groups and the largest size,
rows of one to five entries (matrix in registers) and of six (streamed),
columns at both ends, solves continued over several launches by the server;
against the true residual in float64."""
import numpy as np
import pytest

from paper_2006_14290_amd import synth as S

from gpu_util import dev, host

pytestmark = pytest.mark.gpu

spx = pytest.importorskip("paper_2006_14290_amd.spx")

TOL = 1e-10


def arrow(n, per, seed):
    """Symmetric, diagonally dominant; rows of at most `per` entries, coupled
    to rows far away (first with last)."""
    r = np.random.default_rng(seed)
    D = {}
    deg = np.ones(n, int)
    pairs = [(0, n - 1)] + [tuple(p) for p in r.integers(0, n, (3 * n, 2))]
    for i, j in pairs:
        if i != j and deg[i] < per and deg[j] < per and (i, j) not in D:
            D[i, j] = D[j, i] = -r.uniform(0.5, 1.0)
            deg[i] += 1
            deg[j] += 1
    diag = np.full(n, 0.05)
    for (i, _), v in D.items():
        diag[i] -= v
    for i in range(n):
        D[i, i] = diag[i]
    k = sorted(D)
    rows, cols = np.array([a for a, _ in k]), np.array([b for _, b in k])
    rowptr = np.concatenate([[0], np.cumsum(np.bincount(rows, minlength=n))])
    return S.CSR(n, rowptr.astype(np.int32), cols.astype(np.int32), np.array([D[q] for q in k]))


def check(A, b, x):
    row = np.repeat(np.arange(A.n), np.diff(A.rowptr))
    y, ax = np.zeros(A.n), np.zeros(A.n)
    np.add.at(y, row, A.val * x[A.col])
    np.add.at(ax, row, np.abs(A.val * x[A.col]))
    # the solver's true residual is at most TOL; two evaluations of A x differ
    # by at most eps * |A| |x| per entry of a row
    assert np.linalg.norm(b - y) <= TOL * np.linalg.norm(b) + 2.0 ** -52 * max(8, np.diff(A.rowptr).max()) * np.linalg.norm(ax)


@pytest.mark.parametrize("per", [2, 5, 6])
def test_row_counts(per):
    mats, bs = [], []
    for n in (1, 2, 63, 64, 65, 511, 513, 1023, 1024, 1025, 2049, 3073, 4095, 4096):
        A = arrow(n, per, seed=n + per)
        b = S.uniform_vector(n, seed=n)
        Ad = spx.csr_from_host(A)
        for precond in (0, 1):
            print(f"case n {n} per {per} precond {precond}", flush=True)
            x, info = spx.cg_solve(Ad, dev(b), tol=TOL, maxit=20 * n + 50, precond=precond)
            assert info["status"] == spx.OK
            check(A, b, host(x))
        mats.append((A, Ad))
        bs.append(b)
    print("case batch", flush=True)
    xs, infos = spx.cg_batch([m for _, m in mats], [dev(b) for b in bs], tol=TOL, path=spx.BATCH_ONE_GROUP)
    for (A, _), b, x, info in zip(mats, bs, xs, infos):
        assert info["status"] == spx.OK
        check(A, b, host(x))


def test_continued_over_launches():
    A = arrow(1500, 5, seed=9)
    b = S.uniform_vector(A.n, seed=1)
    xs = []
    for ticks in (1, 1000):
        srv = spx.Server(max_slots=2, hbm_budget_bytes=1 << 26, iters_per_tick=ticks)
        try:
            x, info = srv.wait(srv.submit(A, b, tol=TOL), 60.0)
            assert info["status"] == spx.OK
            xs.append(np.array(x))
        finally:
            srv.close()
    check(A, b, xs[0])
    assert np.array_equal(xs[0], xs[1])


@pytest.mark.parametrize("n", [1, 70, 1000, 3001, 4096])
def test_streamed_rows_of_any_length(n):
    """Rows past the entries in flight: the first row and column full, the
    rest of one to three entries; and every row of about 40."""
    i = np.arange(n)
    D = np.zeros((n, n))
    D[0, 1:] = D[1:, 0] = -0.5 / n
    D[i[1:], i[:-1]] = D[i[:-1], i[1:]] = -0.4
    D[i, i] = 2.0
    r = np.random.default_rng(n)
    M = np.where(r.random((n, n)) < min(1.0, 20 / n), -r.uniform(0.1, 1.0, (n, n)), 0.0)
    M = np.triu(M, 1)
    M = M + M.T
    M[i, i] = 0.1 - M.sum(1)
    for k, dense in (("arrow", D), ("rows of 40", M)):
        rows, cols = np.nonzero(dense)
        A = S.CSR(n, np.concatenate([[0], np.cumsum(np.bincount(rows, minlength=n))]).astype(np.int32),
                  cols.astype(np.int32), dense[rows, cols])
        b = S.uniform_vector(n, seed=n)
        print(f"case {k} n {n}", flush=True)
        x0 = dev(S.uniform_vector(n, seed=n + 1))
        for x in (None, x0):
            x, info = spx.cg_solve(spx.csr_from_host(A), dev(b), x, tol=TOL, maxit=2000)
            assert info["status"] == spx.OK
            check(A, b, host(x))
