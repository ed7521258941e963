"""Launches whose workgroups meet, which later launches tell the host about: the host code (on the CPU), and more launches in
flight than there are units for, on several streams (on the GPU)."""
import os
import shutil
import subprocess

import pytest
import torch

from paper_2601_12698_amd import binding as B
from test_gpu_untuned import bits, norm_inputs
from test_host_sanitizers import BUILD, CSRC, ROOT


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    exe = str(tmp_path_factory.mktemp("tell") / "driver")
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-pthread", "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined", "-Wall",
           "-Wextra", "-I", os.path.join(ROOT, "tests", "fake_hip"), "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-I", BUILD,
           os.path.join(ROOT, "tests", "slot_tell_driver.cpp"), "-o", exe]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=600)
    assert r.returncode == 0, r.stdout[-4000:]
    return exe


@pytest.mark.parametrize("what", ["tells", "tags", "asks", "in_vain", "rotation", "quiet"])
def test_units(driver, what):
    r = subprocess.run([driver, what], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300,
                       env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0"))
    assert r.returncode == 0 and r.stdout.endswith("ok\n"), r.stdout[-4000:]


@pytest.mark.gpu
def test_more_launches_than_units():
    """Three streams with 200 launches of 65 rows, two units each: more than all units, and queued in less time than they take.  Bits
    as where no units are found."""
    B.addrms_table_clear()
    M, N, dtype, launches = 65, 131072, "bf16", 200
    inputs = [norm_inputs(M, N, dtype, 5 * k) for k in range(3)]
    want = []
    for x, _, r, _, w in inputs:
        xw, rw = x.clone(), r.clone()
        for _ in range(launches):
            B.addrms_whole_rows_probe(xw, rw, w, 1e-6, M, N, dtype, False)
        want.append((xw, rw))
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in inputs]
    for _ in range(launches):
        for s, (x, _, r, _, w) in zip(streams, inputs):
            B.addrms_run(x, r, w, 1e-6, M, N, dtype, None, s)
    torch.cuda.synchronize()
    for (x, xok, r, rok, _), (xw, rw) in zip(inputs, want):
        assert torch.equal(bits(x), bits(xw)) and torch.equal(bits(r), bits(rw)) and xok() and rok()
