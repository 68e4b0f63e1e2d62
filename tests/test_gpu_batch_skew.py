"""Small batches of messages of very unlike lengths: many of a few blocks beside
one that makes up most of the bytes, before, after and in the middle of them, and
many tiny ones in an output buffer much larger than they are.  Every result against
the oracle, and the time of the first kind against a batch of as many messages and
bytes, evenly split: no workgroup may end up with all the small messages."""
import numpy as np
import pytest

import oracle
from paper_2007_10752_amd import tdes as T
from paper_2007_10752_amd import workloads as W

pytestmark = pytest.mark.gpu


def _batch(torch, lengths, seed, out_bytes=None):
    g = W.rng(seed)
    lengths = np.asarray(lengths, dtype=np.int64)
    n, total = len(lengths), int(lengths.sum())
    offs = np.concatenate([[0], np.cumsum(lengths)[:-1]]).astype(np.int64)
    keys, dirs = W.key_bundles(g, 61), g.integers(0, 2, size=n).astype(np.uint32)
    idx = g.integers(0, 61, size=n)
    data = W.uniform_bytes(g, total)
    b = T.Batch(keys, offs, offs, lengths, dirs, sched_idx=idx)
    x = torch.from_numpy(data).cuda()
    out = torch.full((out_bytes or total,), 0xA5, dtype=torch.uint8, device="cuda")
    want = data.copy()
    for i in range(n):
        seg = slice(int(offs[i]), int(offs[i] + lengths[i]))
        if lengths[i]:
            want[seg] = oracle.tdes_ecb(keys[idx[i]], data[seg], bool(dirs[i]))
    return b, x, out, want


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


# blocks of the small messages: one each, lengths on both sides of a step's 64th
# part (steps are 64 to 3,072 lanes), some empty
@pytest.mark.parametrize("small", [[1] * 1500, list(range(1, 80)) * 12, [0, 1, 2, 3, 0, 40, 41] * 200])
@pytest.mark.parametrize("where", ["first", "middle", "last", "none"])
def test_unlike_lengths_equal_oracle(torch_dev, small, where):
    blocks = list(small)
    if where != "none":
        blocks.insert({"first": 0, "middle": len(blocks) // 2, "last": len(blocks)}[where], 400_001)
    cus = torch_dev.cuda.get_device_properties(0).multi_processor_count
    # the exact size, or all a small batch's output may hold (1.5 x 2 x 1,024 blocks a CU)
    for out_bytes in (None, 3 * cus * 8192):
        print("skew", len(blocks), where, out_bytes, flush=True)
        b, x, out, want = _batch(torch_dev, np.array(blocks) * 8, W.SEED_BASE + 0x3C0, out_bytes)
        b.submit(x, out)
        torch_dev.cuda.synchronize()
        assert b.skipped() == 0
        got = out.cpu().numpy()
        assert np.array_equal(got[:len(want)], want)
        assert (got[len(want):] == 0xA5).all()


@pytest.mark.parametrize("where", ["first", "last"])
def test_skewed_batch_is_spread_over_the_chip(torch_dev, where):
    # 2,000 messages of a block and one of 5 MB against 2,001 of 2,504 bytes: a few
    # steps more for the small ones, so at most a few times as long (14 times, 482
    # against 34 us, where a single workgroup takes them 64 at a time)
    torch = torch_dev
    skewed = [8] * 2000
    skewed.insert(0 if where == "first" else 2000, 5_000_000)

    def median_us(lengths):
        lengths = np.asarray(lengths, dtype=np.int64)
        offs = np.concatenate([[0], np.cumsum(lengths)[:-1]]).astype(np.int64)
        n = len(lengths)
        b = T.Batch(W.key_bundles(W.rng(W.SEED_BASE), 61), offs, offs, lengths, np.zeros(n, np.uint32),
                    sched_idx=np.arange(n) % 61)
        x = torch.zeros(int(lengths.sum()), dtype=torch.uint8, device="cuda")
        out = torch.empty_like(x)
        times = []
        for i in range(60):
            a, e = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            b.submit(x, out)
            e.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(e) * 1e3)
        return float(np.median(times[20:]))

    even, skew = median_us([2504] * 2001), median_us(skewed)
    print("even", even, "skewed", skew, "us", flush=True)
    assert skew < 5 * even
