"""The scheduler's range allocator used from both ends of the pool, on the host, under
AddressSanitizer and UBSan, against a brute-force model."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_range_alloc_from_both_ends(tmp_path):
    exe = str(tmp_path / "range_alloc_ends_check")
    env = {k: v for k, v in os.environ.items() if k != "LD_PRELOAD"}
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                    "-I", os.path.join(ROOT, "paper_2303_09916_amd", "csrc"),
                    os.path.join(ROOT, "tests", "range_alloc_ends_check.cpp"), "-o", exe], check=True, env=env)
    env["ASAN_OPTIONS"] = "detect_leaks=1"
    r = subprocess.run([exe], capture_output=True, text=True, env=env)
    assert r.returncode == 0, r.stderr
    assert "match the model" in r.stdout
