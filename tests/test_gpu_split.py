"""The bitsliced kernels on both sides of the size up to which a chunk's
S-boxes run on eight waves (five 16 KiB chunks a CU): one block, the edges of
a chunk and of a lane's 16-byte pieces, and above the limit the plain kernel's
last, partial chunk.  Every mode, 16- and 8-byte aligned, bit for bit against
the oracle."""
import numpy as np
import pytest

import oracle
from paper_2007_10752_amd import tdes as T
from paper_2007_10752_amd import workloads as W

pytestmark = pytest.mark.gpu

CHUNK = 16384
# (whole limits of five chunks a CU, bytes beyond)
SIZES = [(0, 8), (0, 1032), (0, CHUNK - 8), (0, CHUNK), (0, CHUNK + 8), (0, 7 * CHUNK + 4104),
         (1, -8), (1, 0), (1, 8), (1, 3 * CHUNK + 264)]


@pytest.mark.parametrize("offset", [0, 8])
@pytest.mark.parametrize("limits,extra", SIZES)
def test_split_and_plain(limits, extra, offset):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    n = limits * 5 * cus * CHUNK + extra
    g = W.rng(W.SEED_BASE + 0x900 + n % 4096)
    key = W.key_bundle(g)
    data = W.uniform_bytes(g, n)
    iv = np.frombuffer((2 ** 64 - 700).to_bytes(8, "big"), np.uint8)  # wraps past block 699
    x = torch.zeros(n + offset, dtype=torch.uint8, device="cuda")[offset:]
    x.copy_(torch.from_numpy(data))
    guard = torch.full((n + offset + 64,), 0xA5, dtype=torch.uint8, device="cuda")
    out = guard[offset: offset + n]
    for name, run, want in (
            ("encrypt", lambda: T.ecb(key, x, out, kernel="bitslice"), oracle.tdes_ecb(key, data)),
            ("decrypt", lambda: T.ecb(key, x, out, decrypt=True, kernel="bitslice"),
             oracle.tdes_ecb(key, data, decrypt=True)),
            ("ctr", lambda: T.ctr(key, iv, x, out), oracle.tdes_ctr(key, iv, data)),
            ("cbc", lambda: T.cbc_decrypt(key, iv, x, out), oracle.tdes_cbc_decrypt(key, iv, data))):
        print(name, n, offset, flush=True)
        out.zero_()
        run()
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy(), want), name
        assert bool((guard[offset + n:] == 0xA5).all()), name  # nothing past the end
    T.ctr(key, iv, x, x)  # in place
    torch.cuda.synchronize()
    assert np.array_equal(x.cpu().numpy(), oracle.tdes_ctr(key, iv, data))
