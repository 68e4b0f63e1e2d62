"""The bitsliced batch kernel, whose batches are small here but go into buffers
past the table kernel's limit: every compiled configuration, in place, at input
offsets past 4 GiB, waves inside one message, and replayed from a captured graph,
bit for bit against the oracle.  Each test checks that this kernel is what runs."""
import numpy as np
import pytest

import oracle
from captured_kernels import kernel_names
from paper_2007_10752_amd import tdes as T
from paper_2007_10752_amd import workloads as W

pytestmark = pytest.mark.gpu

CONFIGS = [(8, 4), (4, 4), (8, 3), (4, 3), (16, 3), (8, 5), (4, 5)]  # as in tdes.h


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


@pytest.fixture(scope="module")
def past_limit(torch_dev):
    # bytes of an output that no batch of up to 2,048 messages leaves to the table kernel
    return 4 * torch_dev.cuda.get_device_properties(0).multi_processor_count * 8192


def _check_kernel(torch, b, x, out):
    names = kernel_names(torch, lambda s: b.submit(x, out, stream=s))
    assert "batch_bitslice_kernel" in names[-1], names


def _want(keys, data, offs, lengths, dirs):
    want = data.copy()
    for i in range(len(lengths)):
        seg = slice(int(offs[i]), int(offs[i] + lengths[i]))
        if lengths[i]:
            want[seg] = oracle.tdes_ecb(keys[i], data[seg], bool(dirs[i]))
    return want


def _offsets(lengths, gap=0):
    return np.concatenate([[0], np.cumsum(np.asarray(lengths) + gap)[:-1]]).astype(np.int64)


# Messages per wave of 64 slices: 64 (lanes widen their own keys), 9 to 20 (on both
# sides of 8- and 16-row tables), 5 to 8, 2 to 4 (4-row tables), and waves inside one
# message (scalar masks), all in one batch, with empty messages between.
def _mixed_lengths(g):
    return np.concatenate([
        g.integers(1, 33, size=200) * 8, [0] * 70, g.integers(97, 225, size=90) * 8,
        g.integers(257, 400, size=60) * 8, [0, 0, 8, 0], g.integers(600, 1100, size=30) * 8,
        [70_008, 16384, 8, 49_160]]).astype(np.int64)


@pytest.mark.parametrize("kmax,waves", CONFIGS)
def test_every_configuration_equals_oracle(torch_dev, past_limit, kmax, waves):
    torch = torch_dev
    g = W.rng(W.SEED_BASE + 0x3E0)
    lengths = _mixed_lengths(g)
    n, total, offs = len(lengths), int(lengths.sum()), _offsets(lengths)
    keys, dirs = W.key_bundles(g, n), g.integers(0, 2, size=n)
    data = W.uniform_bytes(g, total)
    want = _want(keys, data, offs, lengths, dirs)
    x = torch.from_numpy(data).cuda()
    out = torch.empty(past_limit, dtype=torch.uint8, device="cuda")
    b = T.Batch(keys, offs, offs, lengths, dirs)
    keep = T.batch_get_config()
    try:
        for mult in (1, 2, 3, 4):
            T.batch_set_config(kmax, waves, mult)
            _check_kernel(torch, b, x, out)
            print("batch bitslice", kmax, waves, mult, flush=True)
            out.fill_(0xA5)
            b.submit(x, out)
            torch.cuda.synchronize()
            got = out.cpu().numpy()
            assert np.array_equal(got[:total], want), mult
            assert (got[total:] == 0xA5).all(), mult
    finally:
        T.batch_set_config(keep["kmax"], keep["waves"], keep["grid_mult"])


def test_in_place_and_gaps(torch_dev, past_limit):
    torch = torch_dev
    g = W.rng(W.SEED_BASE + 0x3E1)
    lengths = _mixed_lengths(g)
    n, offs = len(lengths), _offsets(lengths, gap=24)
    keys, dirs = W.key_bundles(g, n), g.integers(0, 2, size=n)
    data = W.uniform_bytes(g, past_limit)
    x = torch.from_numpy(data).cuda()
    b = T.Batch(keys, offs, offs, lengths, dirs)
    _check_kernel(torch, b, x, x)
    print("batch bitslice in place", n, flush=True)
    b.submit(x, x)
    torch.cuda.synchronize()
    # (the gaps and everything after the messages stay as they were)
    assert np.array_equal(x.cpu().numpy(), _want(keys, data, offs, lengths, dirs))


def test_waves_inside_one_message(torch_dev, past_limit):
    # whole waves, a wave and a block, odd block counts, one block, at offsets that are
    # multiples of 8 but not of 16, together and each alone
    torch = torch_dev
    g = W.rng(W.SEED_BASE + 0x3E2)
    lengths = np.array([16384, 16392, 3 * 16384 + 8, (1 << 20) + 8, 8, 264, 40, 16, 24,
                        2 * 16384 - 8], dtype=np.int64)
    n, offs = len(lengths), _offsets(lengths, gap=8) + 8
    keys, dirs = W.key_bundles(g, n), g.integers(0, 2, size=n)
    data = W.uniform_bytes(g, past_limit)
    want = _want(keys, data, offs, lengths, dirs)
    x = torch.from_numpy(data).cuda()
    for pick in [slice(0, n)] + [slice(i, i + 1) for i in range(n)]:
        out = x.clone()
        b = T.Batch(keys[pick], offs[pick], offs[pick], lengths[pick], dirs[pick])
        _check_kernel(torch, b, x, out)
        print("batch bitslice one message", pick, flush=True)
        b.submit(x, out)
        torch.cuda.synchronize()
        expect = data.copy()
        for i in range(n)[pick]:
            seg = slice(int(offs[i]), int(offs[i] + lengths[i]))
            expect[seg] = want[seg]
        assert np.array_equal(out.cpu().numpy(), expect), pick


def test_offsets_beyond_4gib(torch_dev, past_limit):
    # input offsets on both sides of byte 2^32 of the base, outputs at low offsets
    torch = torch_dev
    g = W.rng(W.SEED_BASE + 0x3E3)
    lengths = _mixed_lengths(g)
    n, total, rel = len(lengths), int(lengths.sum()), _offsets(lengths)
    keys, dirs = W.key_bundles(g, n), g.integers(0, 2, size=n)
    data = W.uniform_bytes(g, total)
    at = ((1 << 32) - total // 2) & ~7
    x = torch.empty(at + total, dtype=torch.uint8, device="cuda")
    x[at:].copy_(torch.from_numpy(data))
    out = torch.full((past_limit,), 0xA5, dtype=torch.uint8, device="cuda")
    b = T.Batch(keys, at + rel, rel, lengths, dirs)
    _check_kernel(torch, b, x, out)
    print("batch bitslice beyond 4GiB", n, total, at, flush=True)
    b.submit(x, out)
    torch.cuda.synchronize()
    assert b.skipped() == 0
    got = out.cpu().numpy()
    del x, out
    assert np.array_equal(got[:total], _want(keys, data, rel, lengths, dirs))
    assert (got[total:] == 0xA5).all()


@pytest.mark.parametrize("table", [False, True])
def test_graph_replays(torch_dev, past_limit, table):
    # both batch kernels from a captured graph, with new input, eager work and
    # synchronisations between the replays, each against the oracle
    torch = torch_dev
    g = W.rng(W.SEED_BASE + 0x3E4)
    lengths = _mixed_lengths(g)
    n, total, offs = len(lengths), int(lengths.sum()), _offsets(lengths)
    keys, dirs = W.key_bundles(g, n), g.integers(0, 2, size=n)
    x = torch.zeros(total, dtype=torch.uint8, device="cuda")
    out = torch.empty(total if table else past_limit, dtype=torch.uint8, device="cuda")
    b = T.Batch(keys, offs, offs, lengths, dirs)
    names = kernel_names(torch, lambda s: b.submit(x, out, stream=s))
    assert ("batch_table_kernel" if table else "batch_bitslice_kernel") in names[-1], names
    b.submit(x, out)  # eager first: one-time set-up happens outside the capture
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        b.submit(x, out, stream=torch.cuda.current_stream())
    for r in range(3):
        data = W.uniform_bytes(g, total)
        x.copy_(torch.from_numpy(data))
        out.fill_(r)
        torch.cuda.synchronize()
        print("batch graph replay", table, r, flush=True)
        graph.replay()
        torch.cuda.synchronize()
        assert b.skipped() == 0
        got = out.cpu().numpy()
        assert np.array_equal(got[:total], _want(keys, data, offs, lengths, dirs)), r
        assert (got[total:] == r).all()
        eager = torch.full_like(out, 0xA5)
        b.submit(x, eager)
        torch.cuda.synchronize()
        assert torch.equal(eager[:total], out[:total])
