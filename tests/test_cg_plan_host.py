"""The places and the bound of the CG's partials of p.Ap (the kernel header is compiled for the
host with g++ and run on the CPU)."""
import os
import shutil
import subprocess

import pytest

from test_eo_host import CSRC, ROOT, SANITIZE, SANITIZE_ENV


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_partials_cover_every_pair_once_and_are_bounded(tmp_path):
    exe = str(tmp_path / "cg_plan_check")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-Wno-unknown-pragmas", *SANITIZE, "-I", CSRC,
                        "-I", os.path.join(ROOT, "include"), os.path.join(ROOT, "tests", "cg_plan_check.cpp"), "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, env=SANITIZE_ENV)
    assert "Sanitizer" not in r.stderr and "runtime error" not in r.stderr, r.stderr
    assert "FAIL" not in r.stdout, r.stdout
    assert r.returncode == 0, r.stdout
