"""The scalars that end an MCG iteration reach the polling host as pairs of value and tag
(csrc/tagged.h): a read is accepted only when every line of them has arrived, in whatever order
the lines do.  With one tag behind the values the host now and then took the last iteration's
block width, and the solve went wrong."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_partly_arrived_scalars_are_not_read(tmp_path):
    if not shutil.which("g++"):
        pytest.skip("g++ not available")
    exe = str(tmp_path / "tagged")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_2110_04015_amd", "csrc"),
                    os.path.join(ROOT, "tests", "tagged_main.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
