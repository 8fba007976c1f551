"""The length of the server's ticks: a fixed iteration count per tick is for
the systems of one work-group; wide ones follow tick_us, whatever it is."""
import numpy as np
import pytest

import oracle as O
from paper_2006_14290_amd import synth as S

pytestmark = pytest.mark.gpu

spx = pytest.importorskip("paper_2006_14290_amd.spx")


@pytest.mark.parametrize("iters_per_tick", [0, 1, 16])
def test_wide_ticks_follow_tick_us(iters_per_tick):
    print(f"case iters_per_tick={iters_per_tick}", flush=True)
    A = S.poisson2d(1000)
    b = O.csr_spmv(A, S.uniform_vector(A.n, seed=1))
    srv = spx.Server(max_slots=2, hbm_budget_bytes=512 << 20, iters_per_tick=iters_per_tick, tick_us=1_000_000)
    try:
        x, info = srv.wait(srv.submit(A, b, tol=1e-8), timeout_s=60)
        ticks = srv.stats()["ticks"]
    finally:
        srv.close()
    assert info["status"] == spx.OK and info["iters"] > 10 * 96  # more than ten ticks of 96 iterations
    assert np.linalg.norm(b - O.csr_spmv(A, x)) <= 1.01e-8 * np.linalg.norm(b)
    # 512 iterations to a tick once its length is known
    assert ticks <= 4 + info["iters"] // 512, (ticks, info)
