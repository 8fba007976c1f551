"""CSR <-> ELL / HYB / SELL-P at the edges of the 64-row work-groups: sizes
around 64, row lengths around the four parts of a row's slots and the LDS
capacity, hybrid matrices whose COO entries come before, between and after
their slots, padding between slots. Bit for bit against the oracle."""
import numpy as np
import pytest

import oracle as O
from paper_2006_14290_amd import synth as S

from gpu_util import host

pytestmark = pytest.mark.gpu

spx = pytest.importorskip("paper_2006_14290_amd.spx")


def rows_of(n, lo, hi, seed):
    r = np.random.default_rng(seed)
    lens = r.integers(lo, hi + 1, n)
    ncol = max(n, hi)
    col = np.concatenate([np.sort(r.choice(ncol, l, replace=False)) for l in lens]) if n else np.zeros(0)
    rowptr = np.concatenate([[0], np.cumsum(lens)])
    return S.CSR(n, rowptr.astype(np.int32), col.astype(np.int32), r.uniform(-1, 1, rowptr[-1]))


def same(B, A):
    np.testing.assert_array_equal(host(B.rowptr), A.rowptr)
    np.testing.assert_array_equal(host(B.colidx), A.col)
    np.testing.assert_array_equal(host(B.vals).view(np.uint64), A.val.view(np.uint64))


@pytest.mark.parametrize("n", [1, 63, 64, 65, 130])
@pytest.mark.parametrize("lo,hi", [(0, 3), (4, 4), (31, 33), (38, 41), (90, 140)])
def test_round_trips(n, lo, hi):
    print(f"case n={n} {lo}..{hi}", flush=True)
    A = rows_of(n, lo, hi, seed=n + hi)
    Ad = spx.csr_from_host(A)
    E = spx.convert(Ad, spx.ELL, ell_ld=n + 3)
    ref = O.csr_to_ell(A, ld=n + 3)
    np.testing.assert_array_equal(host(E.ell_col), ref.col)
    np.testing.assert_array_equal(host(E.ell_val), ref.val)
    same(spx.convert(E, spx.CSR), A)
    for C, T in ((64, 1), (8, 4), (256, 1)):
        P = spx.convert(Ad, spx.SELLP, slice_size=C, stride_factor=T)
        pref = O.csr_to_sellp(A, C, T)
        np.testing.assert_array_equal(host(P.slice_sets), pref.slice_sets)
        np.testing.assert_array_equal(host(P.ell_col), pref.col)
        np.testing.assert_array_equal(host(P.ell_val), pref.val)
        same(spx.convert(P, spx.CSR), A)
    for K in (0, 1, (lo + hi) // 2):
        H = spx.convert(Ad, spx.HYB, ell_width=K)
        same(spx.convert(H, spx.CSR), A)


@pytest.mark.parametrize("K", [3, 20, 45])
def test_unordered_hybrid_and_inner_padding(K):
    """A random part of every row in COO (before, between and after its
    slots), and padding between slots: still merged in column order."""
    n = 200
    A = rows_of(n, 0, 45, seed=K)
    r = np.random.default_rng(K)
    ecol, eval_ = np.full((K, n), -1, np.int32), np.zeros((K, n))
    crow, ccol, cval = [], [], []
    for i in range(n):
        a, b = A.rowptr[i], A.rowptr[i + 1]
        kept = r.random(b - a) < (0.5 if i % 3 else 1.0)
        idx = np.arange(a, b)[kept][:K]
        slots = np.sort(r.choice(K, idx.size, replace=False))
        ecol[slots, i], eval_[slots, i] = A.col[idx], A.val[idx]
        rest = np.setdiff1d(np.arange(a, b), idx)
        crow += [i] * rest.size
        ccol += list(A.col[rest])
        cval += list(A.val[rest])
    H = spx.hyb_from_host(n, K, n, ecol.reshape(-1), eval_.reshape(-1), np.array(crow), np.array(ccol), np.array(cval))
    same(spx.convert(H, spx.CSR), A)
