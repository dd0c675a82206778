"""The survivor export of the register kernel's tags (pbvd_tag_view.hpp,
compiled for the host) against per-stage decisions, and with every wrong bit
of a tag showing in it."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CXX = shutil.which("g++")


@pytest.mark.skipif(CXX is None, reason="no host compiler")
def test_tag_view(tmp_path):
    exe = str(tmp_path / "tag_view")
    subprocess.run([CXX, "-std=c++17", "-O1", "-Wall", "-Werror", "-I",
                    os.path.join(ROOT, "paper_1608_00066_amd", "csrc"),
                    os.path.join(ROOT, "tests", "native", "tag_view_main.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], stdout=subprocess.PIPE, text=True)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout
