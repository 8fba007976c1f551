"""wave_sum_many on the device (tests/native/wave_sums.hip) for every number of
values: a lane's index below K names the value whose sum over the wavefront it
holds, and every value has such a lane."""
import ctypes
import os

import numpy as np
import pytest
import torch

from gpu_util import dev, host

pytestmark = pytest.mark.gpu

LIB = os.path.join(os.path.dirname(os.path.abspath(__file__)), "native", "libwave_sums.so")


@pytest.mark.parametrize("count", range(1, 65))
def test_sums_and_owners(count):
    print(f"case count={count}", flush=True)
    lib = ctypes.CDLL(LIB)  # build() builds it
    lib.wave_sums.argtypes = [ctypes.c_int] + [ctypes.c_void_p] * 3
    v = np.random.default_rng(count).integers(-(1 << 40), 1 << 40, (count, 64)).astype(np.float64)
    d, total = dev(v), torch.zeros(64, dtype=torch.float64, device="cuda")
    index = torch.zeros(64, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    assert lib.wave_sums(count, d.data_ptr(), total.data_ptr(), index.data_ptr()) == 0
    got, at = host(total), host(index)
    own = at < count
    assert set(at[own]) == set(range(count))
    np.testing.assert_array_equal(got[own], v.sum(1)[at[own]])  # integers: exact in any order
