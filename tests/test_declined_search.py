"""The clustering where the search for partners elsewhere takes no patterns: host code alone, with a search that always declines (host/declined_search.cpp)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(not shutil.which("g++"), reason="needs g++")
def test_the_threads_search_only_where_it_pays_at_their_price(tmp_path):
    exe = str(tmp_path / "declined_search")
    subprocess.run(["g++", "-std=c++17", "-O2", os.path.join(ROOT, "tests", "host", "declined_search.cpp"),
                    os.path.join(ROOT, "paper_2408_11551_amd", "csrc", "preprocess.cpp"), "-o", exe], check=True)
    out = subprocess.run([exe], stdout=subprocess.PIPE, text=True, timeout=100).stdout
    assert out.splitlines()[-1] == "OK", out
