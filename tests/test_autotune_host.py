"""Autotuning keeps the single launch over several shapes unless launches with
tiles were measured faster for that very batch (tests/csrc/autotune_driver.cpp:
the host core against the stand-in runtime, without a GPU)."""
import subprocess

from test_dispatch_host import _build


def test_tiles_of_a_shape_do_not_split_other_batches(tmp_path):
    driver = _build(tmp_path, "autotune_driver.cpp", "ca_api.cpp", "ca_server.cpp")
    r = subprocess.run([str(driver)], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, (r.stdout[-2000:], r.stderr[-4000:])
    assert "ok autotune of shapes" in r.stdout
