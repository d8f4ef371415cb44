"""GPU: the kernels' square root, reciprocal and quotient round correctly, over every float
of their range and some 10^8 pairs; the bits of every search rest on that."""
import os
import re
import subprocess

import pytest

pytestmark = pytest.mark.gpu

EXE = os.path.join(os.path.dirname(os.path.abspath(__file__)), "rounding_check")


def test_roots_reciprocals_and_quotients():
    assert os.path.exists(EXE), "build() makes tests/rounding_check"
    r = subprocess.run([EXE], capture_output=True, text=True, timeout=60)
    print(r.stdout, r.stderr, flush=True)
    got = dict((k, int(v)) for k, v in re.findall(r"(\w+) (\d+)", r.stdout))
    assert r.returncode == 0 and got["floats"] == 102 << 23 and got["pairs"] > 10 ** 8, r.stderr
    assert (got["roots"], got["reciprocals"], got["inverse_roots"], got["quotients"]) == (0, 0, 0, 0)
