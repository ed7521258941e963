"""No two launches with the same place in the memory that workgroups meet in have the same number: the host code of it."""
import os
import shutil
import subprocess

import pytest

from test_host_sanitizers import CSRC, ROOT


def test_numbers_do_not_come_round(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    exe = str(tmp_path / "driver")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined", "-Wall", "-Wextra",
                        "-I", CSRC, os.path.join(ROOT, "tests", "slot_numbers_driver.cpp"), "-o", exe],
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=600)
    assert r.returncode == 0, r.stdout[-4000:]
    r = subprocess.run([exe], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout == "ok\n", r.stdout
