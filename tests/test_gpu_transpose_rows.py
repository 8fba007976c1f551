"""The bucketed CSR transpose with long runs of empty rows: before the first
entry, between two entries, after the last and everywhere; and with exactly as
many entries as its stretches, tiles and segments hold, one less and one more.
Bit for bit against the oracle's counting-sort transpose."""
import numpy as np
import pytest

import oracle as O
from paper_2006_14290_amd import synth as S

from test_gpu_transpose_buckets import check

pytestmark = pytest.mark.gpu

spx = pytest.importorskip("paper_2006_14290_amd.spx")


def exact(n, ncols, nnz, seed, rows=None):
    """n x ncols with exactly nnz distinct entries (in the given rows)."""
    r = np.random.default_rng(seed)
    m = n if rows is None else len(rows)
    assert nnz <= m * ncols
    key = np.empty(0, np.int64)
    while key.size < nnz:
        key = np.unique(np.concatenate([key, r.integers(0, m * ncols, nnz + 64)]))
    key = np.sort(r.permutation(key)[:nnz])
    row = key // ncols if rows is None else np.sort(np.asarray(rows))[key // ncols]
    rowptr = np.zeros(n + 1, np.int64)
    np.add.at(rowptr, row + 1, 1)
    A = S.CSR(n, np.cumsum(rowptr).astype(np.int32), (key % ncols).astype(np.int32), r.uniform(-1, 1, nnz))
    assert A.nnz == nnz == A.rowptr[-1]
    return A


@pytest.mark.parametrize("dtype", ["f64", "f16"])
@pytest.mark.parametrize("n,rows", [
    (300_000, [0]), (300_000, [299_999]), (300_000, [0, 299_999]),
    (300_000, [7, 100_000, 100_001, 250_000]),        # gaps of more rows than a walk takes
    (70_000, list(range(0, 70_000, 35))),              # a gap between any two rows
    (70_000, list(range(100)) + list(range(69_900, 70_000))),
    (5_000, list(range(0, 5_000, 2))), (5_000, list(range(0, 5_000, 3)))])
def test_runs_of_empty_rows(n, rows, dtype):
    for nnz in (len(rows), 1024, 5000):
        if nnz < len(rows):
            continue
        print(f"case n={n} rows={len(rows)} nnz={nnz} {dtype}", flush=True)
        check(exact(n, 6000, nnz, seed=n + nnz, rows=rows), 6000, dtype)


@pytest.mark.parametrize("nnz", [1023, 1024, 1025, 4095, 4096, 4097, 8191, 8192, 8193, 16383, 16384, 16385, 32769])
@pytest.mark.parametrize("ncols", [1, 900, 5000])
def test_entry_counts(nnz, ncols):
    print(f"case nnz={nnz} ncols={ncols}", flush=True)
    check(exact(33_000, ncols, nnz, seed=nnz + ncols), ncols)


@pytest.mark.parametrize("heavy", [16383, 16384, 16385, 2 * 16384 + 1])
def test_segments_of_one_column(heavy):
    """One column of exactly so many entries beside thinly filled ones."""
    print(f"case heavy={heavy}", flush=True)
    n, ncols = 40_000, 4000
    r = np.random.default_rng(heavy)
    rest = np.unique(r.integers(0, n, 9000) * ncols + r.integers(2001, ncols, 9000))
    key = np.sort(np.concatenate([r.choice(n, heavy, replace=False).astype(np.int64) * ncols + 2000, rest]))
    rowptr = np.searchsorted(key, np.arange(n + 1, dtype=np.int64) * ncols)
    A = S.CSR(n, rowptr.astype(np.int32), (key % ncols).astype(np.int32), r.uniform(-1, 1, key.size))
    assert int((A.col == 2000).sum()) == heavy
    check(A, ncols)
