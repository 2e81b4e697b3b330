"""Host checks of csrc/sfmp_schedule.h, which the kernels include: the order of requests and waits of the small-batch form
with streamed activations (no slab is used before it has landed, also if the loads whose values nothing reads are not made),
and the copies of activation blocks (nothing outside a row block is read, whatever counts in the range check)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


def test_requests_and_waits(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / "schedule_driver")
    r = subprocess.run([gxx, "-std=c++17", "-O1", os.path.join(HERE, "schedule_driver.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout == "ok\n", r.stdout + r.stderr
