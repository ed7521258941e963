"""Rows that the registers of one workgroup hold, split over several where they are few: the rule (host code, on the CPU), and the
kernels that may run them (on the GPU)."""
import os
import shutil
import subprocess

import pytest
import torch

from paper_2601_12698_amd import binding as B
from test_gpu_untuned import bits, norm_inputs
from test_host_sanitizers import BUILD, CSRC, HOST_SOURCES, ROOT


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    if not os.path.exists(os.path.join(BUILD, "gen_resources.inc")):
        pytest.skip("the generated instance and resource tables are not present (build the library first)")
    exe = str(tmp_path_factory.mktemp("few") / "driver")
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined", "-Wall", "-Wextra",
           "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-I", BUILD, os.path.join(ROOT, "tests", "few_rows_driver.cpp"),
           *[os.path.join(CSRC, s) for s in HOST_SOURCES + ["direct_route.cpp"]], "-o", exe]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=600)
    assert r.returncode == 0, r.stdout[-4000:]
    return exe


def test_shapes(driver):
    r = subprocess.run([driver, "walk"], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout == "ok\n", r.stdout[-4000:]


LIMITS = [
    (("fp32", 1, 12288), "whole"), (("fp32", 16, 12320), "parts=7 threads=448 pieces=1"), (("fp32", 17, 16384), "whole"),
    (("fp32", 40, 16416), "parts=9 threads=512 pieces=1"), (("fp32", 41, 16416), "whole"), (("fp16_res32", 41, 20480), "whole"),
    (("fp16_res32", 80, 20512), "parts=6 threads=896 pieces=1"), (("fp32", 81, 24576), "whole"),
    (("fp32", 96, 24608), "parts=5 threads=640 pieces=2"), (("fp32", 97, 28672), "whole"),
    (("fp32", 128, 28704), "parts=4 threads=960 pieces=2"), (("fp32", 129, 28704), "whole"),
    (("fp32", 1, 32768), "parts=16 threads=512 pieces=1"), (("bf16", 1, 32768), "whole"), (("fp16", 4, 24576), "whole"),
]


def test_both_sides_of_each_limit(driver):
    lines = "\n".join(f"{B.DTYPE_IDS[d]} {M} {N}" for (d, M, N), _ in LIMITS)
    r = subprocess.run([driver], input=lines, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=120)
    assert r.returncode == 0, r.stdout[-4000:]
    assert [(p, g) for (p, _), g in zip(LIMITS, r.stdout.split("\n"))] == LIMITS


RUNS = {"call": B.addrms_run, "claimed": lambda *a: B.addrms_split_probe(*a, 0), "no units": lambda *a: B.addrms_whole_rows_probe(*a, False),
        "captured": lambda *a: B.addrms_whole_rows_probe(*a, True)}


@pytest.mark.gpu
@pytest.mark.parametrize("run", RUNS)
@pytest.mark.parametrize("dtype,M,N", [("fp32", 16, 12320), ("fp32", 1, 16384), ("fp32", 40, 16417), ("fp16_res32", 3, 32768), ("fp32", 96, 24608),
                                       ("fp16_res32", 128, 32705), ("fp32", 2, 32737), ("fp16_res32", 5, 12291)])
def test_rows(dtype, M, N, run):
    B.addrms_table_clear()
    x, xok, r, rok, w = norm_inputs(M, N, dtype, N)
    xw, rw = x.clone(), r.clone()
    B.addrms_run(xw, rw, w, 1e-6, M, N, dtype, B.addrms_default_cfg(N, dtype))
    RUNS[run](x, r, w, 1e-6, M, N, dtype)
    torch.cuda.synchronize()
    assert torch.equal(bits(r), bits(rw)) and torch.equal(bits(x), bits(xw)) and xok() and rok()
