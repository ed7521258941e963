"""How launches whose workgroups meet say that they are done: the protocol with other threads between any two of its steps (the device
code, compiled for the CPU), and units that come back after every kind of launch (on the GPU)."""
import os
import shutil
import subprocess

import pytest
import torch

from paper_2601_12698_amd import binding as B
from test_gpu_untuned import norm_inputs
from test_host_sanitizers import CSRC, ROOT


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    exe = str(tmp_path_factory.mktemp("report") / "driver")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined", "-Wall", "-Wextra",
                        "-I", os.path.join(ROOT, "tests", "fake_hip"), "-I", CSRC, os.path.join(ROOT, "tests", "unit_report_driver.cpp"), "-o", exe],
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=600)
    assert r.returncode == 0, r.stdout[-4000:]
    return exe


@pytest.mark.parametrize("what", ["pieces", "held_up"])
def test_protocol(driver, what):
    r = subprocess.run([driver, what], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout == "ok\n", r.stdout[-4000:]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,N", [("bf16", 40960), ("fp32", 33001)])
def test_units_come_back(dtype, N):
    """More launches than there are units, each over before the next: one whose end is lost would leave too few of them, and the probe
    takes no other kernel.  Rows that each report in two steps and in one, on either side of eight rows and of a unit."""
    counts = (1, 2, 8, 9, 63, 64, 65, 130)
    x, xok, r, rok, w = norm_inputs(max(counts), N, dtype, 1)
    for i in range(1200):
        M = counts[i % len(counts)]
        B.addrms_split_probe(x[:M * N], r[:M * N], w, 1e-6, M, N, dtype, 256)
        torch.cuda.synchronize()
    assert xok() and rok()
