"""The key expansion that the GPU runs for batches and the server (each lane its own
round key, the schedules' words and the table kernel's keys from it), checked on the
host against the sequential schedule.  Compiled with g++ from
tests/keysched_device_check.cpp."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2007_10752_amd", "csrc")


def test_device_key_expansion_equals_sequential(tmp_path):
    exe = str(tmp_path / "keysched_device_check")
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", CSRC, "-I", os.path.join(ROOT, "include"),
                    "-o", exe, os.path.join(ROOT, "tests", "keysched_device_check.cpp")], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.startswith("ok"), r.stdout + r.stderr


def test_the_kernels_use_it():
    # what the check above compiles is what the two kernels call
    for source, calls in (("batch.hip", ("round_masks(", "schedule_words(")),
                          ("spbox.hip", ("table_round_keys(",))):
        with open(os.path.join(CSRC, source)) as f:
            text = f.read()
        assert all(c in text for c in calls), source
