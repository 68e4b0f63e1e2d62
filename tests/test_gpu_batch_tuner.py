"""The autotuner on a batch that submits run on the table kernel, which no
configuration touches: the current one stays, for single submits and for streams.
The same batch in an output past that kernel's limit is tuned."""
import numpy as np
import pytest

from captured_kernels import kernel_names
from paper_2007_10752_amd import tdes as T
from paper_2007_10752_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [40, 2500])  # scanned by the kernel itself, and not
@pytest.mark.parametrize("config", [(4, 5, 4), (16, 3, 1)])
def test_small_batches_leave_the_configuration(n, config, tmp_path, monkeypatch):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    monkeypatch.setenv("TDES_TUNE_CACHE", str(tmp_path / "tune.json"))
    g = W.rng(W.SEED_BASE + 0x3D0 + n)
    lengths = (g.integers(1, 40, size=n) * 8).astype(np.int64)
    offs = np.concatenate([[0], np.cumsum(lengths)[:-1]]).astype(np.int64)
    total = int(lengths.sum())
    x = torch.from_numpy(W.uniform_bytes(g, total)).cuda()
    b = T.Batch(W.key_bundles(g, n), offs, offs, lengths, g.integers(0, 2, size=n))
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    outs = [torch.empty(total, dtype=torch.uint8, device="cuda") for _ in range(2)]
    large = torch.empty(4 * cus * 8192, dtype=torch.uint8, device="cuda")
    keep = T.batch_get_config()
    try:
        assert "batch_table" in kernel_names(torch, lambda s: b.submit(x, outs[0], stream=s))[-1]
        assert "batch_bitslice" in kernel_names(torch, lambda s: b.submit(x, large, stream=s))[-1]
        b.submit(x, outs[0])
        torch.cuda.synchronize()
        want = outs[0].clone()
        for tune in (lambda: b.autotune(x, outs[0], reps=3),
                     lambda: b.autotune_streams(x, outs, [torch.cuda.Stream(), torch.cuda.Stream()],
                                                reps=3)):
            T.batch_set_config(*config)
            print("tune", n, config, flush=True)
            m = tune()
            assert (m["kmax"], m["waves"], m["grid_mult"], m["saved"]) == config + (1,)
            cur = T.batch_get_config()
            assert (cur["kmax"], cur["waves"], cur["grid_mult"]) == config
        torch.cuda.synchronize()
        assert all(torch.equal(o, want) for o in outs)
        other = torch.empty_like(large)
        for tune in (lambda: b.autotune(x, large, reps=1),
                     lambda: b.autotune_streams(x, [large, other],
                                                [torch.cuda.Stream(), torch.cuda.Stream()], reps=1)):
            m = tune()
            torch.cuda.synchronize()
            cur = T.batch_get_config()
            assert all(cur[k] == m[k] for k in ("kmax", "waves", "grid_mult"))
        assert torch.equal(large[:total], want) and torch.equal(other[:total], want)
    finally:
        T.batch_set_config(keep["kmax"], keep["waves"], keep["grid_mult"])
