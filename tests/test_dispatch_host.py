"""Batches of several frame shapes are dispatched as such by every route -- a
cached plan, the entry point without allocation, a server -- and for every
scorer, also where the shapes have one area (tests/csrc/dispatch_driver.cpp:
the host core against the stand-in runtime, without a GPU)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_2210_14771_amd", "csrc")


def _build(tmp_path, driver, *sources):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    out = tmp_path / "driver"
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined",
           "-fno-sanitize-recover=all", "-I", os.path.join(HERE, "csrc", "hip_stub"),
           "-I", os.path.join(HERE, "csrc"), "-I", os.path.join(ROOT, "include"), "-I", CSRC,
           os.path.join(HERE, "csrc", driver), *[os.path.join(CSRC, s) for s in sources],
           "-o", str(out)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    return out


def test_shapes_are_dispatched_alike_by_every_route(tmp_path):
    driver = _build(tmp_path, "dispatch_driver.cpp", "ca_api.cpp", "ca_server.cpp")
    r = subprocess.run([str(driver)], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, (r.stdout[-2000:], r.stderr[-4000:])
    assert "ok dispatch of shapes" in r.stdout
