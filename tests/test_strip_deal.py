"""The learned scorers' strips are divided by their real work: every wave's share
replayed on the CPU (tests/csrc/deal_driver.cpp) covers each position once, and
the last wave's steps stay near the mean for batches of any size."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2210_14771_amd", "csrc")


def test_waves_shares_are_even(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    out = tmp_path / "deal"
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined",
                        "-fno-sanitize-recover=all", "-I", CSRC,
                        os.path.join(HERE, "csrc", "deal_driver.cpp"), "-o", str(out)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([str(out)], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, (r.stdout[-2000:], r.stderr[-4000:])
    assert "ok deal" in r.stdout
