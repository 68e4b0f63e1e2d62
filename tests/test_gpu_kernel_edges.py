"""Key bundles at the edges of the key material, in-place, 8-byte aligned, ragged
and side-stream calls on each ECB kernel, at sizes that it takes: the groups of
eight lanes, the table kernel with a block a lane, the split and the plain bitsliced
kernel.  The data repeat a run of blocks, so that the oracle's result on the run is
the whole answer.  Each test checks that the kernel it names is what runs."""
import numpy as np
import pytest

import oracle
from captured_kernels import kernel_names
from paper_2007_10752_amd import tdes as T
from paper_2007_10752_amd import workloads as W

pytestmark = pytest.mark.gpu

# kernel: (choice, name in its mangled name, blocks a CU, blocks beyond)
KERNELS = {
    "group": ("spbox", "tdes_spbox_group_kernel", 100, 5),
    "table": ("spbox", "17tdes_spbox_kernel", 130, 77),
    "table, several blocks a lane": ("spbox", "17tdes_spbox_kernel", 4 * 4096 + 3 * 1024, 321),
    "split": ("bitslice", "tdes_bitslice_split_kernel", 2048, 1234),
    "plain": ("bitslice", "20tdes_bitslice_kernel", 5 * 2048, 2048 + 1237),
}
RUN = 4099  # blocks that repeat: no divisor of a lane's, a wave's or a chunk's blocks


def _bundles():
    g = W.rng(W.SEED_BASE + 0x3F0)
    k = [W.key_bundle(g)[:8] for _ in range(3)]
    weak = lambda h: np.tile(np.frombuffer(bytes.fromhex(h), np.uint8), 3)
    return {
        "zero": np.zeros(24, np.uint8), "ones": np.full(24, 0xFF, np.uint8),
        "weak_01": weak("0101010101010101"), "weak_fe": weak("FEFEFEFEFEFEFEFE"),
        "weak_e0": weak("E0E0E0E0F1F1F1F1"), "weak_1f": weak("1F1F1F1F0E0E0E0E"),
        "single": np.concatenate([k[0], k[0], k[0]]),
        "k1_eq_k2": np.concatenate([k[0], k[0], k[1]]),
        "two_key": np.concatenate([k[0], k[1], k[0]]), "three_key": np.concatenate(k),
    }


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _repeated(torch, run, nblk):
    r = torch.from_numpy(run).cuda()
    return r.repeat(-(-nblk // RUN))[:8 * nblk]


def _setup(torch, kernel, offset=0):
    choice, name, per_cu, extra = KERNELS[kernel]
    nblk = per_cu * torch.cuda.get_device_properties(0).multi_processor_count + extra
    run = W.uniform_bytes(W.rng(W.SEED_BASE + 0x3F1), 8 * RUN)
    x = torch.empty(8 * nblk + offset, dtype=torch.uint8, device="cuda")[offset:]
    x.copy_(_repeated(torch, run, nblk))
    names = kernel_names(torch, lambda s: T.ecb(bytes(24), x, x, False, choice, s))
    assert len(names) == 1 and name in names[0], names
    return choice, nblk, run, x


@pytest.mark.parametrize("kernel", list(KERNELS))
@pytest.mark.parametrize("bundle", list(_bundles()))
def test_edge_bundles(torch_dev, kernel, bundle):
    torch = torch_dev
    key = _bundles()[bundle]
    choice, nblk, run, x = _setup(torch, kernel)
    for dec in (False, True):
        print("edge", kernel, bundle, dec, nblk, flush=True)
        out = T.ecb(key, x, None, dec, choice)
        torch.cuda.synchronize()
        assert torch.equal(out, _repeated(torch, oracle.tdes_ecb(key, run, dec), nblk)), dec


@pytest.mark.parametrize("kernel", list(KERNELS))
@pytest.mark.parametrize("offset,inplace", [(8, False), (0, True), (8, True)])
def test_unaligned_and_in_place(torch_dev, kernel, offset, inplace):
    torch = torch_dev
    choice, nblk, run, x = _setup(torch, kernel, offset)
    key = W.key_bundle(W.rng(W.SEED_BASE + 0x3F2))
    print("unaligned or in place", kernel, offset, inplace, nblk, flush=True)
    guard = torch.full((8 * nblk + offset + 64,), 0xA5, dtype=torch.uint8, device="cuda")
    out = x if inplace else guard[offset:offset + 8 * nblk]
    T.ecb(key, x, out, False, choice)
    torch.cuda.synchronize()
    assert torch.equal(out, _repeated(torch, oracle.tdes_ecb(key, run), nblk))
    assert bool((guard[offset + 8 * nblk:] == 0xA5).all())


@pytest.mark.parametrize("kernel", list(KERNELS))
def test_side_stream(torch_dev, kernel):
    torch = torch_dev
    choice, nblk, run, x = _setup(torch, kernel)
    key = W.key_bundle(W.rng(W.SEED_BASE + 0x3F3))
    out, back = torch.zeros_like(x), torch.zeros_like(x)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    print("side stream", kernel, nblk, flush=True)
    T.encrypt(key, x, out, kernel=choice, stream=s)
    T.decrypt(key, out, back, kernel=choice, stream=s)
    s.synchronize()
    assert torch.equal(out, _repeated(torch, oracle.tdes_ecb(key, run), nblk))
    assert torch.equal(back, x)
