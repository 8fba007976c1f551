"""Hybrid matrices whose slots are not in column order, to CSR: the slots keep
their order, and each is preceded by the COO entries, in theirs, that lie
below it and have not been placed."""
import numpy as np
import pytest

from gpu_util import host

pytestmark = pytest.mark.gpu

spx = pytest.importorskip("paper_2006_14290_amd.spx")


@pytest.mark.parametrize("K", [2, 3, 9, 40])
def test_slots_out_of_order(K):
    print(f"case K={K}", flush=True)
    n, ncoo = 200, 5
    r = np.random.default_rng(K)
    ecol, eval_ = np.full((K, n), -1, np.int32), np.zeros((K, n))
    crow, ccol, cval, want = [], [], [], []
    for i in range(n):
        slots = r.integers(0, K + 1)
        cols = r.choice(n, slots + ncoo, replace=False)
        vals = r.uniform(-1, 1, slots + ncoo)
        if i % 4 == 0:  # the last slot is below the first COO entry, another one above it
            cols[:slots] = np.sort(cols[:slots])[::-1]
        ecol[:slots, i], eval_[:slots, i] = cols[:slots], vals[:slots]
        o = slots + np.argsort(cols[slots:])
        crow += [i] * ncoo
        ccol += list(cols[o])
        cval += list(vals[o])
        left = list(o)
        for k in range(slots):
            while left and cols[left[0]] < cols[k]:
                want.append((cols[left[0]], vals[left.pop(0)]))
            want.append((cols[k], vals[k]))
        want += [(cols[q], vals[q]) for q in left]
    H = spx.hyb_from_host(n, K, n, ecol.reshape(-1), eval_.reshape(-1), np.array(crow), np.array(ccol), np.array(cval))
    C = spx.convert(H, spx.CSR)
    np.testing.assert_array_equal(host(C.colidx), np.array([c for c, _ in want], np.int32))
    np.testing.assert_array_equal(host(C.vals), np.array([v for _, v in want]))
