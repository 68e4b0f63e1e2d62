"""Which kernel an ECB call runs: the explicit choices the kernel they name at
every size, the automatic choice the one tdes_ecb_auto_kernel answers with.  The
calls are captured, not run."""
import pytest

from captured_kernels import kernel_names
from paper_2007_10752_amd import tdes as T

pytestmark = pytest.mark.gpu

KiB, MiB = 1 << 10, 1 << 20
NAME = {"spbox": "tdes_spbox", "bitslice": "tdes_bitslice"}


# (bytes a CU, bytes beyond): around the limits of the eight-lane groups (1 KiB a
# CU), of a workgroup of the table kernel a CU (8 KiB), of the automatic choice (24
# KiB) and of the split kernel (five chunks of 16 KiB)
@pytest.mark.parametrize("per_cu,extra", [(0, 8), (0, 32 * KiB), (1 * KiB, 0), (1 * KiB, 8),
                                          (8 * KiB, 0), (8 * KiB, 8), (16 * KiB, 0), (24 * KiB, -8),
                                          (24 * KiB, 0), (24 * KiB, 8), (80 * KiB, 0),
                                          (80 * KiB, 8), (0, 64 * MiB)])
def test_kernel_of_an_ecb_call(per_cu, extra):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n = per_cu * torch.cuda.get_device_properties(0).multi_processor_count + extra
    x = torch.empty(n, dtype=torch.uint8, device="cuda")
    for kernel in ("auto", "spbox", "bitslice"):
        for decrypt in (False, True):
            names = kernel_names(torch, lambda s: T.ecb(bytes(24), x, x, decrypt, kernel, s))
            want = T.auto_kernel(n) if kernel == "auto" else kernel
            print(n, kernel, names, flush=True)
            assert len(names) == 1 and NAME[want] in names[0], (n, kernel, want, names)
