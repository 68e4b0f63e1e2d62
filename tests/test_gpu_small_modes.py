"""CTR and CBC decryption on both sides of the table kernel's limit (its
workgroups one to a CU) and of the limit up to which eight lanes share a block
(128 blocks a CU), and around a workgroup of such groups (32 blocks), in place
and 8-byte aligned, bit for bit against the oracle; ECB's automatic choice at
the same sizes."""
import numpy as np
import pytest

import oracle
from paper_2007_10752_amd import tdes as T
from paper_2007_10752_amd import workloads as W

pytestmark = pytest.mark.gpu


# (blocks per CU, blocks beyond)
@pytest.mark.parametrize("per_cu,extra", [(0, 1), (0, 31), (0, 32), (0, 33), (128, 0), (128, 1),
                                          (1024, -1), (1024, 0), (1024, 1)])
@pytest.mark.parametrize("offset", [0, 8])
def test_modes_around_the_table_kernels_limit(per_cu, extra, offset):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    n = 8 * (per_cu * cus + extra)
    g = W.rng(W.SEED_BASE + 0x980 + n % 4096)
    key, iv = W.key_bundle(g), np.frombuffer((2 ** 64 - 40).to_bytes(8, "big"), np.uint8)
    data = W.uniform_bytes(g, n)
    x = torch.zeros(n + offset, dtype=torch.uint8, device="cuda")[offset:]
    x.copy_(torch.from_numpy(data))
    guard = torch.full((n + offset + 64,), 0xA5, dtype=torch.uint8, device="cuda")
    out = guard[offset: offset + n]
    for name, run, want in (
            ("ecb", lambda: T.encrypt(key, x, out), oracle.tdes_ecb(key, data)),
            ("ctr", lambda: T.ctr(key, iv, x, out), oracle.tdes_ctr(key, iv, data)),
            ("cbc", lambda: T.cbc_decrypt(key, iv, x, out), oracle.tdes_cbc_decrypt(key, iv, data))):
        print(name, n, offset, flush=True)
        run()
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy(), want), name
        assert bool((guard[offset + n:] == 0xA5).all()), name
    T.ctr(key, iv, x, x)
    torch.cuda.synchronize()
    assert np.array_equal(x.cpu().numpy(), oracle.tdes_ctr(key, iv, data))
