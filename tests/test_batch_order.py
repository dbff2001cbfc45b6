"""Order of a batch call's table upload against earlier work on the same table, on
the CPU: tests/cpp/batch_order_test.cpp with the library's own batch.cpp against a
model of HIP's queues (tests/cpp/fake_hip)."""
from __future__ import annotations

import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_2607_02630_amd", "csrc")


@pytest.mark.parametrize("scenario", ["handles", "failures"])
def test_uploads_wait_for_every_reader_of_the_table(tmp_path, scenario):
    exe = tmp_path / "batch_order_test"
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-pthread", "-I", os.path.join(HERE, "cpp", "fake_hip"), "-I", CSRC,
                    "-o", str(exe), os.path.join(HERE, "cpp", "batch_order_test.cpp"),
                    *(os.path.join(CSRC, f) for f in ("batch.cpp", "host_pool.cpp", "keys.cpp", "tune.cpp")), "-ldl"],
                   check=True)
    r = subprocess.run([str(exe), scenario], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "batch order ok" in r.stdout, r.stdout + r.stderr
