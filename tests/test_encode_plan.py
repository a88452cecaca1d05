"""What the encode decisions ask for, and the outputs that may not lie over it (CPU, g++)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not found")
def test_requests_and_overlaps(tmp_path):
    exe = str(tmp_path / "encode_plan")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-Wall", "-fsanitize=undefined", "-fno-sanitize-recover=all",
                           os.path.join(HERE, "plan", "encode_plan_main.cpp"), "-o", exe])
    r = subprocess.run([exe], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-3000:]
