"""The bucketed CSR transpose at its edges, bit for bit against the oracle's
counting-sort transpose: entry counts around its tiles and segments, column
counts around its bucket widths and beyond them (the radix sort), heavy
columns that need several segments, runs of empty rows, every value width."""
import numpy as np
import pytest

import oracle as O
from paper_2006_14290_amd import synth as S

from gpu_util import host

pytestmark = pytest.mark.gpu

spx = pytest.importorskip("paper_2006_14290_amd.spx")


def random_rect(n, ncols, nnz, seed, heavy=None):
    """n x ncols with about nnz distinct entries; `heavy`: columns that hold
    half of them."""
    r = np.random.default_rng(seed)
    col = r.integers(0, ncols, nnz)
    if heavy is not None:
        half = r.random(nnz) < 0.5
        col[half] = np.asarray(heavy)[r.integers(0, len(heavy), int(half.sum()))]
    row = r.integers(0, n, nnz)
    row[row % 7 < 3] = n // 2  # runs of empty rows beside one long row
    key = np.unique(row.astype(np.int64) * ncols + col)
    rowptr = np.searchsorted(key, np.arange(n + 1, dtype=np.int64) * ncols)
    return S.CSR(n, rowptr.astype(np.int32), (key % ncols).astype(np.int32), r.uniform(-1, 1, key.size))


def check(A, ncols, dtype="f64"):
    Ad = spx.csr_from_host(A, spx.DTYPE_NAMES[dtype])
    Ad.ncols = ncols
    At = spx.csr_transpose(Ad)
    rp, col, val = O.csr_transpose(A, ncols=ncols)
    np.testing.assert_array_equal(host(At.rowptr), rp)
    np.testing.assert_array_equal(host(At.colidx)[:A.nnz], col)
    stored = val.astype({"f64": np.float64, "f32": np.float32, "f16": np.float16}[dtype])
    np.testing.assert_array_equal(host(At.vals)[:A.nnz].view(np.uint8), stored.view(np.uint8))


@pytest.mark.parametrize("nnz", [1, 63, 64, 2047, 2049, 8192, 8193, 40000, 300000])
@pytest.mark.parametrize("ncols", [1, 2, 1024, 1025, 5000])
def test_sizes(nnz, ncols):
    print(f"case nnz={nnz} ncols={ncols}", flush=True)
    check(random_rect(3000, ncols, nnz, seed=nnz + ncols), ncols)


@pytest.mark.parametrize("ncols", [1 << 21, (1 << 21) + 1, 3_000_000, 1 << 22, (1 << 22) + 1])
def test_many_columns(ncols):
    print(f"case ncols={ncols}", flush=True)
    check(random_rect(5000, ncols, 200_000, seed=3), ncols)


@pytest.mark.parametrize("dtype", ["f64", "f32", "f16"])
@pytest.mark.parametrize("heavy", [[4096], [0, 1, 2], [9999]])
def test_heavy_columns(heavy, dtype):
    """Buckets far above one segment, at both ends and in the middle."""
    print(f"case heavy={heavy} {dtype}", flush=True)
    check(random_rect(400_000, 10_000, 700_000, seed=4, heavy=heavy), 10_000, dtype)


def test_banded_and_single_column():
    check(S.poisson3d_7pt(40), 64_000)
    n = 100_000
    one = S.CSR(n, np.arange(n + 1, dtype=np.int32), np.zeros(n, np.int32), np.arange(n, dtype=np.float64))
    check(one, 1)
