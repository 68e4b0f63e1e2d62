"""The batched table kernel and the batched bitsliced kernel on the same
batches, bit for bit against the oracle.  Which one runs depends on the output
buffer's size: exact-sized outputs take the table kernel here, the same batch
into a large buffer the bitsliced one.  Batches at the edges: one block; as many
messages as a workgroup holds round keys for, and one more; as many as it scans
itself, and one more; long runs of empty messages; invalid messages."""
import numpy as np
import pytest

import oracle
from paper_2007_10752_amd import tdes as T
from paper_2007_10752_amd import workloads as W

pytestmark = pytest.mark.gpu


def _lengths(kind, g):
    if kind == "one block":
        return [8]
    if kind.startswith("blocks "):  # one-block messages
        return [8] * int(kind.split()[1])
    if kind.startswith("tiny "):
        return g.integers(0, 25, size=int(kind.split()[1])) * 8
    if kind == "empty runs":  # more empty messages in a row than are staged at once
        return np.concatenate([[16], [0] * 1500, [8, 0, 24], [0] * 1024, g.integers(1, 9, size=900) * 8,
                               [0] * 1023, [64], [0] * 5])
    if kind == "long":
        return [200_008, 8, 1 << 20, 72, 400_000]
    return np.maximum(8, np.ceil(g.lognormal(8.3, 1.0, size=300) / 8) * 8)


@pytest.mark.parametrize("kind", ["one block", "blocks 64", "blocks 65", "blocks 1030", "tiny 2048",
                                  "tiny 2049", "tiny 6000", "empty runs", "long", "mixed 300"])
def test_table_and_bitsliced_batches(kind):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    g = W.rng(W.SEED_BASE + 0x3A0 + len(kind))
    lengths = np.asarray(_lengths(kind, g), dtype=np.int64)
    n, total = len(lengths), int(lengths.sum())
    offs = np.concatenate([[0], np.cumsum(lengths)[:-1]]).astype(np.int64)
    keys, dirs = W.key_bundles(g, 97), g.integers(0, 2, size=n).astype(np.uint32)
    idx = g.integers(0, 97, size=n)
    data = W.uniform_bytes(g, total)
    want = data.copy()
    for i in range(n):
        seg = slice(int(offs[i]), int(offs[i] + lengths[i]))
        if lengths[i]:
            want[seg] = oracle.tdes_ecb(keys[idx[i]], data[seg], bool(dirs[i]))
    bad = None
    if n > 40:  # a message past the buffer: skipped, its place left alone
        bad = int(np.flatnonzero(lengths)[20])
        want[int(offs[bad]):int(offs[bad] + lengths[bad])] = 0xA5
    x = torch.from_numpy(data).cuda()
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    large = max(4 * cus * 8192, 2048 * n)  # past both limits of the table kernel
    for out_bytes, configs in ((total, [(8, 4, 2)]), (large, [(8, 4, 2), (4, 3, 1), (16, 3, 4)])):
        for cfg in configs:
            T.batch_set_config(*cfg)
            out = torch.full((out_bytes,), 0xA5, dtype=torch.uint8, device="cuda")
            b = T.Batch(keys, offs, offs, lengths, dirs, sched_idx=idx)
            if bad is not None:
                b.msgs[bad, 1] = 1 << 40
            print(kind, out_bytes, cfg, flush=True)
            for repeat in range(2):
                b.submit(x, out)
            torch.cuda.synchronize()
            assert b.skipped() == (bad is not None)
            got = out.cpu().numpy()
            assert np.array_equal(got[:total], want), cfg
            assert bool((got[total:] == 0xA5).all()), cfg
            skipped = torch.zeros(1, dtype=torch.int64, device="cuda")
            out.fill_(0xA5)
            T.batch_submit_noalloc_ptr(b.msgs.data_ptr(), n, b.sched.data_ptr(), b.n_sched,
                                       x.data_ptr(), total, out.data_ptr(), out_bytes,
                                       skipped.data_ptr(), b.stream)
            torch.cuda.synchronize()
            assert int(skipped.item()) == (bad is not None)
            assert np.array_equal(out.cpu().numpy()[:total], want), cfg
    T.batch_set_config(8, 4, 2)


@pytest.mark.parametrize("n, blocks_per_cu", [(3, 1023), (40, 1025), (300, 2049), (2048, 1100), (5, 3072)])
def test_several_blocks_a_lane(n, blocks_per_cu):
    # Around the sizes at which a lane takes one, two or three blocks of a batch.
    # (The oracle checks each message's ends and a part in its middle, the plain
    # kernel the whole of it.)
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    total = 8 * (blocks_per_cu * cus - 3)
    g = W.rng(W.SEED_BASE + 0x3B0 + n)
    cuts = np.sort(g.choice(total // 8 - 1, size=n - 1, replace=False) + 1)
    starts = np.concatenate([[0], cuts]).astype(np.int64) * 8
    lengths = np.diff(np.concatenate([starts, [total]]))
    keys, dirs = W.key_bundles(g, n), g.integers(0, 2, size=n).astype(np.uint32)
    data = W.uniform_bytes(g, total)
    x = torch.from_numpy(data).cuda()
    out, ref = torch.full_like(x, 0xA5), torch.empty_like(x)
    b = T.Batch(keys, starts, starts, lengths, dirs)
    b.submit(x, out)
    for i in range(n):
        seg = slice(int(starts[i]), int(starts[i] + lengths[i]))
        T.ecb(bytes(keys[i]), x[seg], ref[seg], decrypt=bool(dirs[i]), kernel="bitslice")
    torch.cuda.synchronize()
    assert b.skipped() == 0
    assert torch.equal(out, ref)
    got = out.cpu().numpy()
    for i in g.choice(n, size=min(n, 24), replace=False):
        for at in (0, int(lengths[i]) // 16 * 8, max(0, int(lengths[i]) - 64)):
            seg = slice(int(starts[i]) + at, int(starts[i]) + min(at + 64, int(lengths[i])))
            assert np.array_equal(got[seg], oracle.tdes_ecb(keys[i], data[seg], bool(dirs[i]))), (i, at)
