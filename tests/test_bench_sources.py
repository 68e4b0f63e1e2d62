"""The source hash that stored counter readings are matched by covers every file a
kernel is compiled from: an edit to any file that the compiler reads for it (its own
list of dependencies) changes the hash."""
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)


@pytest.mark.parametrize("kernel", ["bitslice", "spbox"])
def test_source_hash_follows_every_dependency(tmp_path, monkeypatch, kernel):
    import bench
    from paper_2007_10752_amd import build
    if not os.path.exists(build.HIPCC):
        pytest.skip("no hipcc")
    csrc = tmp_path / "paper_2007_10752_amd" / "csrc"
    shutil.copytree(build.CSRC, csrc)
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    r = subprocess.run([build.HIPCC, "-MM", "-std=c++17", "-x", "hip", "--cuda-host-only",
                        "-I", os.path.join(ROOT, "include"), "-I", str(csrc),
                        str(csrc / (kernel + ".hip"))], capture_output=True, text=True, check=True)
    deps = [d for d in r.stdout.replace("\\\n", " ").split()[1:] if d.startswith(str(csrc))]
    assert len(deps) > 3, r.stdout
    whole = bench.kernel_source_hash(kernel)
    for d in deps:
        with open(d) as f:
            text = f.read()
        with open(d, "a") as f:
            f.write("\n// edited\n")
        assert bench.kernel_source_hash(kernel) != whole, d
        with open(d, "w") as f:
            f.write(text)
    assert bench.kernel_source_hash(kernel) == whole
