"""The decoders' LDS exchange (tests/layout_x4d_check.cpp, compiled
with g++): every coordinate found where it was put, no bank conflicts."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_lds_exchange_of_the_decoders(tmp_path):
    exe = str(tmp_path / "layout_x4d_check")
    subprocess.run(["g++", "-O1", "-std=c++17", f"-I{os.path.join(ROOT, 'paper_2407_01378_amd', 'csrc')}", "-o", exe,
                    os.path.join(ROOT, "tests", "layout_x4d_check.cpp")], check=True)
    res = subprocess.run([exe], stdout=subprocess.PIPE, text=True)
    assert res.returncode == 0 and "0 problems" in res.stdout, res.stdout
