"""The split of a small box's maps into runs (the most costly run as cheap as can be,
with the fewest runs), on the host, against every other split."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_map_runs(tmp_path):
    exe = str(tmp_path / "map_runs_check")
    env = {k: v for k, v in os.environ.items() if k != "LD_PRELOAD"}
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                    "-I", os.path.join(ROOT, "paper_2303_09916_amd", "csrc"),
                    os.path.join(ROOT, "tests", "map_runs_check.cpp"), "-o", exe], check=True, env=env)
    r = subprocess.run([exe], capture_output=True, text=True, env=env)
    assert r.returncode == 0, r.stderr
    assert "as specified" in r.stdout
