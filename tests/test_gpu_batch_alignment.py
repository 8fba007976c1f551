"""A wide batched system's solution does not depend on where its arrays lie:
bit for bit the same from arrays that 16-byte copies can read and from arrays
that they cannot, alone and in a batch, for rows of every staged class."""
import numpy as np
import pytest

from test_gpu_batch_stage import device, spd_band

from gpu_util import dev, host

pytestmark = pytest.mark.gpu

spx = pytest.importorskip("paper_2006_14290_amd.spx")


@pytest.mark.parametrize("n,half", [(9000, 2), (9001, 3), (8193, 7), (5000, 15), (4999, 31), (4200, 60)])
def test_bits(n, half):
    print(f"case n={n} half={half}", flush=True)
    A = spd_band(n, half, seed=n + half)
    b = np.random.default_rng(half).uniform(-1, 1, n)
    mats = [device(A, shift) for shift in (0, 1, 2, 3)]
    assert {m.vals.data_ptr() % 16 for m in mats} == {0, 8} and {m.colidx.data_ptr() % 16 for m in mats} == {0, 4, 8, 12}
    alone, info = zip(*(spx.cg_batch([m], [dev(b)], tol=1e-10) for m in mats))
    mixed, _ = spx.cg_batch(mats, [dev(b)] * 4, tol=1e-10)
    first = host(alone[0][0])
    for x in [a[0] for a in alone[1:]] + list(mixed):
        np.testing.assert_array_equal(host(x).view(np.uint64), first.view(np.uint64))
