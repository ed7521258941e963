"""Configured launches whose outputs are written through to the memory-side cache: which they are (on the CPU), and that they
are what an ordinary store leaves, on either side of each limit (on the GPU)."""
import os
import shutil
import subprocess

import pytest
import torch

from paper_2601_12698_amd import binding as B
from test_gpu_untuned import bits, finite, norm_inputs
from test_host_sanitizers import BUILD, CSRC, HOST_SOURCES, ROOT

NORM, SILU, MERGE = 0, 1, 2
LIMITS = [  # op, dtype, N, cfg, fewest and most rows
    (NORM, "bf16", 4096, "8,512,1,0,1,2,0,0", 1221, 6144), (NORM, "bf16", 4096, "8,256,2,0,2,3,0,0", 1221, 6144),
    (NORM, "bf16", 4096, "2,512,1,1,4,34,0,0", 1221, 6144), (NORM, "bf16", 7168, "8,448,1,0,1,34,6,0", 698, 3510),
    (NORM, "fp16", 512, "8,64,2,0,1,2,0,0", 9766, 49152), (NORM, "fp16_res32", 5120, "2,512,1,0,2,34,0,0", 652, 3276),
    (NORM, "fp16_res32", 2880, "4,384,1,0,2,2,0,0", 1158, 5825), (NORM, "fp16_res32", 1024, "8,128,1,0,1,2,0,0", 3256, 16384),
    (NORM, "fp16_res32", 1000, "4,64,16,0,4,98,0,0", 3334, 16777), (NORM, "fp32", 8192, "4,1024,1,0,2,2,0,0", 306, 1536),
    (SILU, "bf16", 11008, "8,704,1,0,1,2,0,0", 1817, 4572), (SILU, "fp32", 4096, "4,512,1,0,2,3,0,0", 2442, 6144),
    (SILU, "fp16", 4096, "2,512,1,0,4,2,0,0", 4883, 12288)]
NEVER = [
    (NORM, "bf16", 4000, 4096, "8,512,1,0,1,0,0,0"), (NORM, "bf16", 4000, 4096, "8,512,1,0,1,6,0,0"),
    (NORM, "bf16", 4000, 4104, "8,576,1,0,1,2,0,0"), (NORM, "fp16", 4000, 4096, "1,1024,1,0,4,2,0,0"),
    (SILU, "bf16", 4000, 8192, "8,1024,1,0,1,0,0,0"), (SILU, "bf16", 4000, 8200, "8,1024,1,0,1,2,0,0"),
    (MERGE, "bf16", 100000, 256, "8,32,8,0,1,2,0,0"),
    # instances without that kind of store: more than six chunks, one element per chunk, forms for long rows
    (NORM, "bf16", 2000, 8192, "2,512,1,0,1,2,0,0"), (NORM, "fp32", 3000, 4096, "1,1024,1,0,4,2,0,0"),
    (SILU, "fp32", 3000, 4096, "1,1024,1,0,4,2,0,0"), (NORM, "bf16", 400, 40960, "8,1024,1,0,2,18,0,0"), (NORM, "bf16", 400, 40960, "8,1024,1,0,2,10,0,0")]


def test_which_launches_write_through(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    if not os.path.exists(os.path.join(BUILD, "gen_resources.inc")):
        pytest.skip("the generated instance and resource tables are not present (build the library first)")
    exe = str(tmp_path / "driver")
    cmd = ["g++", "-std=c++17", "-O1", "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined", "-Wall", "-Wextra",
           "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-I", BUILD, os.path.join(ROOT, "tests", "write_through_driver.cpp"),
           *[os.path.join(CSRC, s) for s in HOST_SOURCES], "-o", exe]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=600)
    assert r.returncode == 0, r.stdout[-4000:]
    lines = [(op, dt, M, N, cfg) for op, dt, N, cfg, lo, hi in LIMITS for M in (lo - 1, lo, hi, hi + 1)] + NEVER
    r = subprocess.run([exe], input="\n".join(f"{op} {B.DTYPE_IDS[dt]} {M} {N} {cfg}" for op, dt, M, N, cfg in lines),
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=120)
    assert r.returncode == 0, r.stdout[-4000:]
    assert r.stdout.split() == ["0", "1", "1", "0"] * len(LIMITS) + ["0"] * len(NEVER)


@pytest.mark.parametrize("what", ["chooses", "layouts", "general", "accepted"])
def test_store_kinds_in_a_search(what, tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    if not os.path.exists(os.path.join(BUILD, "gen_resources.inc")):
        pytest.skip("the generated instance and resource tables are not present (build the library first)")
    exe = str(tmp_path / "driver")
    cmd = ["g++", "-std=c++17", "-O1", "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined", "-Wall", "-Wextra",
           "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-I", BUILD, os.path.join(ROOT, "tests", "store_kinds_driver.cpp"),
           *[os.path.join(CSRC, s) for s in HOST_SOURCES], "-o", exe]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=600)
    assert r.returncode == 0, r.stdout[-4000:]
    r = subprocess.run([exe, what], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout == "ok\n", r.stdout[-4000:]


def test_a_saved_kind_of_store_comes_back(tmp_path):
    B.addrms_table_clear()
    cfg = B.make_cfg(4, 64, 16, 0, 4, B.FLAG_NONTEMPORAL | B.FLAG_DEFER_STORE | B.FLAG_ALIGNED_SPAN | B.FLAG_STREAM_STORES)
    B.addrms_table_insert(8192, 1000, "fp16_res32", cfg, 17.6)
    B.addrms_table_save(str(tmp_path / "t"))
    B.addrms_table_clear()
    B.addrms_table_load(str(tmp_path / "t"))
    assert B.addrms_table_lookup(8192, 1000, "fp16_res32").as_tuple() == cfg.as_tuple()
    B.addrms_table_clear()


@pytest.mark.gpu
@pytest.mark.parametrize("op,dtype,M,N,plan", [(NORM, "fp16_res32", 8192, 1000, "4,64,16,0,4,98,0,0"), (NORM, "bf16", 2633, 7168, "8,448,1,0,1,34,6,0"),
                                               (SILU, "bf16", 4000, 11008, "8,704,1,0,1,2,0,0")])
def test_results_with_either_kind_of_store(op, dtype, M, N, plan):
    through, stream = (B.Cfg(*map(int, plan.split(","))) for _ in range(2))
    stream.flags |= B.FLAG_STREAM_STORES
    x, xok, r, rok, w = norm_inputs(M, 2 * N if op == SILU else N, dtype, 5)
    if op == NORM:
        xw, rw = x.clone(), r.clone()
        B.addrms_run(xw, rw, w, 1e-6, M, N, dtype, through)
        B.addrms_run(x, r, w, 1e-6, M, N, dtype, stream)
        torch.cuda.synchronize()
        assert torch.equal(bits(x), bits(xw)) and torch.equal(bits(r), bits(rw)) and xok() and rok()
    else:
        a, b = (torch.ones(M, N, dtype=x.dtype, device="cuda") for _ in range(2))
        B.silumul_run(x, a, M, N, dtype, through)
        B.silumul_run(x, b, M, N, dtype, stream)
        torch.cuda.synchronize()
        assert torch.equal(bits(a), bits(b))


@pytest.mark.gpu
@pytest.mark.parametrize("at", ["below", "fewest", "most"])
@pytest.mark.parametrize("op,dtype,N,plan,lo,hi", LIMITS)
def test_results_on_both_sides(op, dtype, N, plan, lo, hi, at):
    M = {"below": lo - 1, "fewest": lo, "most": hi}[at]
    cfg = B.Cfg(*map(int, plan.split(",")))
    ordinary = B.Cfg(*map(int, plan.split(",")))                  # the same shape, and ordinary stores
    ordinary.flags &= ~2
    if op == NORM:
        x, xok, r, rok, w = norm_inputs(M, N, dtype, 3)
        xw, rw = x.clone(), r.clone()
        B.addrms_run(xw, rw, w, 1e-6, M, N, dtype, ordinary)
        B.addrms_run(x, r, w, 1e-6, M, N, dtype, cfg)
        torch.cuda.synchronize()
        assert torch.equal(bits(x), bits(xw)) and torch.equal(bits(r), bits(rw)) and xok() and rok()
    else:
        t = {"bf16": torch.bfloat16, "fp16": torch.float16, "fp32": torch.float32}[dtype]
        x = finite((M, 2 * N), t, 4)
        guard = torch.full((M + 2, N), 7.0, dtype=t, device="cuda")
        out, want = guard[1:-1], torch.ones(M, N, dtype=t, device="cuda")
        B.silumul_run(x, want, M, N, dtype, ordinary)
        B.silumul_run(x, out, M, N, dtype, cfg)
        torch.cuda.synchronize()
        assert torch.equal(bits(out), bits(want)) and bool((guard[0] == 7).all()) and bool((guard[-1] == 7).all())
