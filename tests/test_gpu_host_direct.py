"""Direct host-resident ECB at the edges of its launch shapes: one block, the
switches between the workgroups' working lanes, one block per lane of every CU
and the steps beyond; in place and with a guard behind the output, bit for bit
against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2007_10752_amd import tdes as T
from paper_2007_10752_amd import workloads as W

pytestmark = pytest.mark.gpu


# (blocks per CU, blocks beyond)
@pytest.mark.parametrize("per_cu,extra", [(0, 1), (64, -1), (64, 1), (1024, 0), (1024, 1), (2048, 77)])
def test_direct_launch_shapes(per_cu, extra):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n = 8 * (per_cu * torch.cuda.get_device_properties(0).multi_processor_count + extra)
    g = W.rng(W.SEED_BASE + 0x9C0 + n % 4096)
    key, data = W.key_bundle(g), W.uniform_bytes(g, n)
    x = torch.empty(n, dtype=torch.uint8, pin_memory=True)
    x.numpy()[:] = data
    guard = torch.empty(n + 64, dtype=torch.uint8, pin_memory=True)
    guard.fill_(0xA5)
    print("direct", n, flush=True)
    T.ecb_host(key, x, guard[:n])
    want = oracle.tdes_ecb(key, data)
    assert np.array_equal(guard.numpy()[:n], want)
    assert bool((guard[n:] == 0xA5).all())
    T.ecb_host(key, x, x)
    assert np.array_equal(x.numpy(), want)
    T.ecb_host(key, x, x, decrypt=True)
    assert np.array_equal(x.numpy(), data)
