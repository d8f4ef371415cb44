"""The host construction of the pair stream (a layout of the intra-ligand term) against
a plain construction, at atom and pair counts around its chunks, and its cost: it is
part of every scoring call, so it must not go through every list for every chunk."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
@pytest.mark.parametrize("flags", [["-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all"], ["-O2", "-DTIMED"]])
def test_pair_stream_construction(tmp_path, flags):
    exe = str(tmp_path / "pair_stream_check")
    env = {k: v for k, v in os.environ.items() if k != "LD_PRELOAD"}
    subprocess.run(["g++", "-std=c++17", *flags, "-I", os.path.join(ROOT, "paper_2303_09916_amd", "csrc"),
                    os.path.join(ROOT, "tests", "pair_stream_check.cpp"), "-o", exe], check=True, env=env)
    r = subprocess.run([exe], capture_output=True, text=True, env=env)
    print(r.stdout)
    assert r.returncode == 0, r.stderr
    assert "as specified" in r.stdout
