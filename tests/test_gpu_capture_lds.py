"""An eager call of long rows prepares the kernel that the same call takes in a capture: the limit of its LDS is raised then
(and its code object loaded), and the capture makes no such call.  In a process of its own, where nothing has raised it yet, with hipFuncSetAttribute
replaced by one that counts and passes on."""
import os
import shutil
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SHIM = """
static int (*real)(const void*, int, int);
static int calls;
void shim_pass_on_to(void* f) { real = (int (*)(const void*, int, int))f; }
int shim_calls(void) { return calls; }
int hipFuncSetAttribute(const void* fn, int attr, int value) { ++calls; return real(fn, attr, value); }
"""

CHILD = """
import ctypes, os, sys
shim = ctypes.CDLL(sys.argv[1], ctypes.RTLD_GLOBAL)       # before the library is loaded, which then finds the shim's
import torch
hip = ctypes.CDLL(os.path.join(os.path.dirname(torch.__file__), "lib", "libamdhip64.so"))
shim.shim_pass_on_to(ctypes.cast(hip.hipFuncSetAttribute, ctypes.c_void_p))
from paper_2601_12698_amd import binding as B
M, N = 3, int(sys.argv[2])
x, r = (torch.ones(M, N, device="cuda", dtype=torch.bfloat16) for _ in range(2))
w = torch.ones(N, device="cuda", dtype=torch.bfloat16)
torch.cuda.synchronize()
start = shim.shim_calls()
B.addrms_run(x, r, w, 1e-6, M, N, "bf16")
torch.cuda.synchronize()
eager = shim.shim_calls()
graph = torch.cuda.CUDAGraph()
with torch.cuda.graph(graph):
    begin = shim.shim_calls()
    B.addrms_run(x, r, w, 1e-6, M, N, "bf16")
    end = shim.shim_calls()
graph.replay()
torch.cuda.synchronize()
print("calls", eager - start, end - begin, flush=True)
"""


@pytest.mark.parametrize("N", [81920, 40960])                   # 128 KB of LDS, and none
def test_an_eager_call_raises_the_limit_for_captures(tmp_path, N):
    if shutil.which("gcc") is None:
        pytest.skip("no gcc")
    src, so = tmp_path / "shim.c", str(tmp_path / "shim.so")
    src.write_text(SHIM)
    subprocess.run(["gcc", "-shared", "-fPIC", "-O1", "-o", so, str(src)], check=True, timeout=60)
    r = subprocess.run([sys.executable, "-c", CHILD, so, str(N)], cwd=ROOT, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True,
                       timeout=110)
    assert r.returncode == 0, r.stdout[-4000:]
    assert r.stdout.strip().endswith("calls 1 0"), r.stdout[-4000:]
