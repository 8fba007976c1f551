"""The float32 sums of the staged-rows CSR product are no further from float64
than a tree over the row's rounded products (the order of one lane per entry)."""
import numpy as np
import pytest

from paper_2006_14290_amd import synth as S

from gpu_util import dev, host

pytestmark = pytest.mark.gpu

spx = pytest.importorskip("paper_2006_14290_amd.spx")


def tree(A, val, x, width):
    """Row sums of float32 products, halved from `width` padded lanes on."""
    lens = np.diff(A.rowptr)
    k = np.arange(width)
    on = k < lens[:, None]
    e = np.where(on, A.rowptr[:-1, None] + k, 0)
    p = np.where(on, val[e] * x[A.col[e]], np.float32(0)).astype(np.float32)
    while p.shape[1] > 1:
        p = p[:, : p.shape[1] // 2] + p[:, p.shape[1] // 2:]
    return p[:, 0].astype(np.float64)


@pytest.mark.parametrize("name,width", [("7-point", 8), ("27-point", 32)])
def test_error_of_float32_sums(name, width):
    print(f"case {name}", flush=True)
    A = S.poisson3d_7pt(50) if name == "7-point" else S.stencil27_random(30, seed=3)
    val = A.val.astype(np.float32)
    x = S.uniform_vector(A.n, seed=4).astype(np.float32)
    exact = np.add.reduceat(val.astype(np.float64) * x.astype(np.float64)[A.col], A.rowptr[:-1])
    y = host(spx.spmv(spx.csr_from_host(A, spx.F32), dev(x))).astype(np.float64)
    err, bar = (np.linalg.norm(v - exact) / np.linalg.norm(exact) for v in (y, tree(A, val, x, width)))
    print(f"error {err:.4g}, tree {bar:.4g}", flush=True)
    assert err <= bar
