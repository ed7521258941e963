"""Configured launches whose waves wait for one load before they ask for more: which they are (on the CPU), and that it makes
no difference to the results on either side of each limit (on the GPU)."""
import os
import shutil
import subprocess

import pytest
import torch

from paper_2601_12698_amd import binding as B
from test_gpu_untuned import bits, finite, norm_inputs
from test_host_sanitizers import BUILD, CSRC, HOST_SOURCES, ROOT

NORM, SILU, MERGE = 0, 1, 2
LIMITS = [  # op, dtype, M that is not, N, cfg: one row more is paced
    (NORM, "bf16", 6103, 4096, "8,512,1,0,1,0,0,0"), (NORM, "bf16", 6103, 4096, "8,256,1,0,2,32,0,0"),
    (NORM, "fp16_res32", 4068, 4096, "4,512,1,0,2,0,0,0"), (NORM, "fp32", 3051, 4096, "4,512,1,0,2,0,0,0"),
    (SILU, "bf16", 1953, 4096, "8,512,1,0,1,2,0,0"), (SILU, "fp32", 976, 4096, "4,512,1,0,1,2,0,0"),
    (SILU, "bf16", 32552, 4096, "8,512,1,0,1,0,0,0"), (SILU, "fp16", 32552, 4096, "8,256,1,0,2,2,0,0")]
NEVER = [
    (NORM, "bf16", 200000, 4096, "8,512,1,0,1,2,0,0"), (NORM, "bf16", 200000, 7168, "8,448,1,0,1,34,6,0"),
    (NORM, "bf16", 200000, 4096, "8,512,1,0,1,1,0,0"), (NORM, "bf16", 200000, 4096, "8,512,1,0,1,4,0,0"),
    (NORM, "bf16", 200000, 4096, "8,512,1,0,1,0,6,0"), (NORM, "fp16", 200000, 4095, "1,512,1,0,4,0,0,0"),
    (NORM, "fp16_res32", 200000, 4096, "2,512,1,0,2,0,0,0"), (SILU, "bf16", 200000, 8192, "8,1024,1,0,1,3,0,0"),
    (SILU, "bf16", 200000, 4100, "4,512,1,0,2,2,0,0"), (SILU, "fp32", 200000, 4098, "2,512,1,0,2,0,0,0"),
    (MERGE, "bf16", 10000000, 256, "8,32,8,0,1,0,0,0")]


def test_which_launches_are_paced(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    if not os.path.exists(os.path.join(BUILD, "gen_resources.inc")):
        pytest.skip("the generated instance and resource tables are not present (build the library first)")
    exe = str(tmp_path / "driver")
    cmd = ["g++", "-std=c++17", "-O1", "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined", "-Wall", "-Wextra",
           "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-I", BUILD, os.path.join(ROOT, "tests", "paced_driver.cpp"),
           *[os.path.join(CSRC, s) for s in HOST_SOURCES], "-o", exe]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=600)
    assert r.returncode == 0, r.stdout[-4000:]
    lines = [(op, dt, M + more, N, cfg) for op, dt, M, N, cfg in LIMITS for more in (0, 1)] + NEVER
    r = subprocess.run([exe], input="\n".join(f"{op} {B.DTYPE_IDS[dt]} {M} {N} {cfg}" for op, dt, M, N, cfg in lines),
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=120)
    assert r.returncode == 0, r.stdout[-4000:]
    assert r.stdout.split() == ["0", "1"] * len(LIMITS) + ["0"] * len(NEVER)


@pytest.mark.gpu
@pytest.mark.parametrize("more", [0, 1])
@pytest.mark.parametrize("op,dtype,M,N,plan", LIMITS)
def test_results_on_both_sides(op, dtype, M, N, plan, more):
    cfg, M = B.Cfg(*map(int, plan.split(","))), M + more
    capped = B.Cfg(*map(int, plan.split(",")))                    # the same kernel, and never paced
    capped.max_waves_per_simd = 4
    if op == NORM:
        x, xok, r, rok, w = norm_inputs(M, N, dtype, 3)
        xw, rw = x.clone(), r.clone()
        B.addrms_run(xw, rw, w, 1e-6, M, N, dtype, capped)
        B.addrms_run(x, r, w, 1e-6, M, N, dtype, cfg)
        torch.cuda.synchronize()
        assert torch.equal(bits(x), bits(xw)) and torch.equal(bits(r), bits(rw)) and xok() and rok()
    else:
        t = {"bf16": torch.bfloat16, "fp16": torch.float16, "fp32": torch.float32}[dtype]
        x = finite((M, 2 * N), t, 4)
        out, want = torch.zeros(M, N, dtype=t, device="cuda"), torch.ones(M, N, dtype=t, device="cuda")
        B.silumul_run(x, want, M, N, dtype, capped)
        B.silumul_run(x, out, M, N, dtype, cfg)
        torch.cuda.synchronize()
        assert torch.equal(bits(out), bits(want))
