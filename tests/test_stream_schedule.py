"""The order of requests and waits of the small-batch form with streamed activations (csrc/sfmp_stream_schedule.h, which the
kernel includes), run on the host against a model of the memory queue: no slab is used before it has landed, also if the
loads whose values nothing reads are not made."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


def test_no_slab_is_used_before_it_has_landed(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / "stream_schedule_driver")
    r = subprocess.run([gxx, "-std=c++17", "-O1", os.path.join(HERE, "stream_schedule_driver.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout == "ok\n", r.stdout + r.stderr
