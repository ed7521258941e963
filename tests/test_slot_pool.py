"""Which launches may use the same piece of the memory that workgroups meet in: the host code of it, on the CPU."""
import os
import shutil
import subprocess

import pytest

from test_host_sanitizers import BUILD, CSRC, ROOT


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    exe = str(tmp_path_factory.mktemp("slots") / "driver")
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-pthread", "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined", "-Wall",
           "-Wextra", "-I", os.path.join(ROOT, "tests", "fake_hip"), "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-I", BUILD,
           os.path.join(ROOT, "tests", "slot_pool_driver.cpp"), "-o", exe]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=600)
    assert r.returncode == 0, r.stdout[-4000:]
    return exe


@pytest.mark.parametrize("what", ["devices", "handles", "leases", "waiting", "errors"])
def test_units_of_launches_in_flight(driver, what):
    r = subprocess.run([driver, what], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300,
                       env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0"))
    assert r.returncode == 0 and r.stdout.endswith("ok\n"), r.stdout[-4000:]
