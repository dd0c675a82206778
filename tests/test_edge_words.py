"""The words through which blocks exchange the bits of a byte they share do not
depend on what earlier calls left in them (pbvd_edges.hpp, compiled for the
host)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CXX = shutil.which("g++")


@pytest.mark.skipif(CXX is None, reason="no host compiler")
def test_edge_words(tmp_path):
    exe = str(tmp_path / "edge_words")
    subprocess.run([CXX, "-std=c++17", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_1608_00066_amd", "csrc"),
                    os.path.join(ROOT, "tests", "native", "edge_words_main.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], stdout=subprocess.PIPE, text=True)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout
