"""The COO product where rows cross the wavefronts' spans: a first row that
closes in the first tile, at a tile's or a chunk's end or not at all, rows over
several spans, single entries at a span's ends; plain and as the COO part of
a hybrid matrix, against the CPU oracle."""
import numpy as np
import pytest

import oracle as O
from paper_2006_14290_amd import synth as S

from gpu_util import assert_spmv_f64, assert_spmv_low, dev, host

pytestmark = pytest.mark.gpu

spx = pytest.importorskip("paper_2006_14290_amd.spx")

CHUNK = 256  # entries of a span of a small matrix


def from_lengths(lens, seed):
    r = np.random.default_rng(seed)
    n = len(lens)
    rowptr = np.concatenate([[0], np.cumsum(lens)])
    col = np.concatenate([np.sort(r.choice(n, k, replace=False)) for k in lens])
    return S.CSR(n, rowptr.astype(np.int32), col.astype(np.int32), r.uniform(-1, 1, rowptr[-1]))


def pattern(name):
    n = 6000
    r = np.random.default_rng(7)
    if name == "ones":
        return np.ones(n, int)
    if name == "tile ends":  # rows that end at multiples of 64 entries, shifted by one now and then
        return np.concatenate([np.resize([63, 1, 64, 65, 63], 200), np.ones(n - 200, int)])
    if name == "chunk ends":
        return np.concatenate([np.resize([CHUNK - 1, 1, CHUNK, CHUNK + 1, CHUNK - 1, 2 * CHUNK, 3], 120),
                               np.zeros(n - 120, int)])
    if name == "long":  # several whole spans, first, in the middle and last
        lens = r.integers(0, 6, n)
        lens[[0, 1, n // 2, n - 1]] = [5 * CHUNK + 7, CHUNK, 4 * CHUNK, 3 * CHUNK - 1]
        return lens
    return r.integers(0, 60, n)


@pytest.mark.parametrize("dtype", ["f64", "f32", "f16"])
@pytest.mark.parametrize("name", ["ones", "tile ends", "chunk ends", "long", "ragged"])
def test_rows_across_spans(name, dtype):
    print(f"case {name} {dtype}", flush=True)
    A = from_lengths(pattern(name), seed=len(name))
    vec = np.float64 if dtype == "f64" else np.float32
    stored = A.val.astype({"f64": np.float64, "f32": np.float32, "f16": np.float16}[dtype]).astype(np.float64)
    x = S.uniform_vector(A.n, seed=1).astype(vec).astype(np.float64)
    y0 = S.uniform_vector(A.n, seed=2).astype(vec).astype(np.float64)
    Ad = spx.csr_from_host(A, spx.DTYPE_NAMES[dtype])
    for M in (spx.convert(Ad, spx.COO), spx.convert(Ad, spx.HYB, ell_width=0), spx.convert(Ad, spx.HYB, ell_width=1)):
        for alpha, beta in ((1.0, 0.0), (-1.5, 0.5)):
            yref, absax = O.csr_spmv_dot2(S.CSR(A.n, A.rowptr, A.col, stored), x, y0, alpha=alpha, beta=beta)
            y = host(spx.spmv(M, dev(x, M.vec_dtype), dev(y0, M.vec_dtype), alpha=alpha, beta=beta))
            if dtype == "f64":
                assert_spmv_f64(y, yref, abs(alpha) * absax, beta_y=beta * y0)
            else:
                assert_spmv_low(y, yref, abs(alpha) * absax, np.diff(A.rowptr), beta_y=beta * y0)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_large_chunks(dtype):
    """2^25 entries and more in the COO part: larger chunks where x fits an
    L2 (float32), tile by tile where it does not (float64), stored and
    accumulated, with and without beta."""
    per, n = 35, (1 << 20) - 17
    print(f"case {dtype}", flush=True)
    off = np.sort(np.random.default_rng(per).choice(4 * per, per, replace=False))
    col = np.minimum(np.arange(n)[:, None], n - 4 * per) + off
    A = S.CSR(n, (np.arange(n + 1) * per).astype(np.int32), col.reshape(-1).astype(np.int32),
              np.random.default_rng(1).uniform(-1, 1, n * per))
    vec = np.float64 if dtype == "f64" else np.float32
    stored = A.val.astype(vec).astype(np.float64)
    x = S.uniform_vector(n, seed=1).astype(vec).astype(np.float64)
    y0 = S.uniform_vector(n, seed=2).astype(vec).astype(np.float64)
    Ad = spx.csr_from_host(A, spx.DTYPE_NAMES[dtype])
    hyb, coo = spx.convert(Ad, spx.HYB, ell_width=1), spx.convert(Ad, spx.COO)
    assert hyb.coo_nnz >= 1 << 25 and coo.nnz >= 1 << 25
    for alpha, beta in ((1.0, 0.0), (-1.5, 0.5)):
        yref, absax = O.csr_spmv_dot2(S.CSR(n, A.rowptr, A.col, stored), x, y0, alpha=alpha, beta=beta)
        for M in (hyb, coo):
            y = host(spx.spmv(M, dev(x, M.vec_dtype), dev(y0, M.vec_dtype), alpha=alpha, beta=beta))
            if dtype == "f64":
                assert_spmv_f64(y, yref, abs(alpha) * absax, beta_y=beta * y0)
            else:
                assert_spmv_low(y, yref, abs(alpha) * absax, np.diff(A.rowptr), beta_y=beta * y0)
