"""The dense estimate's search in the list of selected chunks (topkc_search.h) against the position it has by
construction, for lists of every length up to the largest that the entry points take (2^32 - 1 entries, where 32-bit
sums of positions come round), and the mark of a chunk that is not in it.  The check is a small C++ program (tests/topkc_search_check.cpp) compiled with g++."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_search_in_the_list_of_selected_chunks(tmp_path):
    exe = str(tmp_path / "topkc_search_check")
    src = os.path.join(ROOT, "tests", "topkc_search_check.cpp")
    inc = os.path.join(ROOT, "paper_2407_01378_amd", "csrc")
    subprocess.run(["g++", "-O1", "-std=c++17", f"-I{inc}", "-o", exe, src], check=True)
    res = subprocess.run([exe], stdout=subprocess.PIPE, text=True)
    assert res.returncode == 0, res.stdout
    assert "0 problems" in res.stdout
