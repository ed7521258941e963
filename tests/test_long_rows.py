"""Long rows without a configuration by each of the three kernels that may run them: split over workgroups (eager calls), one
workgroup that parks in LDS what its registers do not hold and reads the rest twice (captured calls), and one workgroup that
forms the split's sums (eager calls that find no memory for the workgroups to meet in)."""
import pytest
import torch

from paper_2601_12698_amd import binding as B
from paper_2601_12698_amd import workloads as W
from test_gpu_untuned import LONG, bits, norm_inputs
from test_split_rows import SPLIT
from test_split_rows import driver as split_driver          # noqa: F401
from test_untuned_route import driver as route_driver       # noqa: F401
from test_untuned_route import routes

# formats, policies and numbers of pieces that neither list has
MORE = [("fp16", 450, 57344), ("fp16", 300, 99991), ("fp32", 150, 100001), ("fp16_res32", 200, 86016), ("bf16", 2, 131071),
        ("fp16", 33, 131008), ("fp16_res32", 2, 86016), ("bf16", 70, 121401), ("fp16", 70, 121401), ("fp16_res32", 90, 86016),
        ("fp32", 60, 131072), ("fp32", 3, 32800), ("fp16", 400, 57344)]
WHOLE = ("bf16", 1, 1 << 20)                                      # in LONG, and not split
CASES = sorted({*LONG, *SPLIT, *MORE} - {WHOLE, ("bf16", 700, 40960)})


def test_the_cases_run_every_kernel(split_driver, route_driver):  # noqa: F811
    import subprocess
    lines = "\n".join(f"{B.DTYPE_IDS[d]} {M} {N}" for d, M, N in CASES)
    r = subprocess.run([split_driver], input=lines, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=120)
    assert r.returncode == 0, r.stdout[-4000:]
    long, split, alone, parts = set(), set(), set(), set()
    for (dtype, _, N), s, l in zip(CASES, r.stdout.split("\n"), routes(route_driver, [("addrms", *c) for c in CASES])):
        assert s != "whole" and l.startswith("long"), (dtype, N, s, l)
        ragged, pieces = "ragged" in l, s.split("pieces=")[1].split()[0]
        long.add((dtype, l.split()[1], ragged))
        split.add((dtype, pieces, s.split()[-1], ragged))
        alone.add((dtype, pieces, ragged))
        vec, parked = (8 if dtype in ("bf16", "fp16") else 4), int(l.split("parked=")[1])
        parts.add((dtype, parked > 0, N > 1024 * (48 + vec * (parked + 1))))
    assert len(long) == 4 * 2 * 2 and len(split) == 4 * 4 * 2 and len(alone) == 4 * 3 * 2
    assert parts == {(d, *p) for d in W.DTYPES for p in ((False, False), (True, False), (True, True))}   # parked, read twice


def check(run, M, N, dtype, off=0, special=None, weight_off=0):
    x, xok, r, rok, w = norm_inputs(M, N, dtype, N, off, special)
    if weight_off:
        w = torch.cat([w[:weight_off], w])[weight_off:]
    xw, rw = x.clone(), r.clone()
    if off:                                                       # the clones start at an aligned address
        xw, rw = torch.cat([xw[:off], xw])[off:], torch.cat([rw[:off], rw])[off:]
    B.addrms_run(xw, rw, w, 1e-6, M, N, dtype, B.addrms_default_cfg(N, dtype))
    run(x, r, w, 1e-6, M, N, dtype)
    torch.cuda.synchronize()
    assert torch.equal(bits(r), bits(rw)) and torch.equal(bits(x), bits(xw)) and xok() and rok()


KERNELS = {"split": lambda *a: B.addrms_split_probe(*a, 256), "captured": lambda *a: B.addrms_whole_rows_probe(*a, True),
           "no units": lambda *a: B.addrms_whole_rows_probe(*a, False)}
kernels = pytest.mark.parametrize("kernel", KERNELS)


@pytest.mark.gpu
@kernels
@pytest.mark.parametrize("dtype,M,N", CASES)
def test_bits_of_the_default_configuration(kernel, dtype, M, N):
    check(KERNELS[kernel], M, N, dtype)


@pytest.mark.gpu
@kernels
@pytest.mark.parametrize("dtype", W.DTYPES)
@pytest.mark.parametrize("N", [33000, 86019, 131072])
def test_infinities_and_nan_stay_in_their_rows(kernel, dtype, N):
    inf = float("inf")
    check(KERNELS[kernel], 7, N, dtype, special=[(1, 0, inf), (3, N // 2, -inf), (4, N - 1, inf), (5, N - 1, float("nan"))])


@pytest.mark.gpu
@kernels
@pytest.mark.parametrize("off", [1, 3])
def test_ragged_rows_from_any_element(kernel, off):
    for dtype in W.DTYPES:
        check(KERNELS[kernel], 3, 40001, dtype, off)
        check(KERNELS[kernel], 3, 90001, dtype, off)


@pytest.mark.gpu
@kernels
@pytest.mark.parametrize("dtype", W.DTYPES)
def test_bases_that_only_a_narrow_default_access_fits(kernel, dtype):
    """86912: as in test_gpu_untuned.py, whole vectors whose default configuration reads two elements at a time
    (and, at more than 1 MB, leaves them to these kernels)."""
    assert B.addrms_default_cfg(86912, dtype).vec < (8 if dtype in ("bf16", "fp16") else 4)
    for off in (0, 2, 4, 6):
        check(KERNELS[kernel], 4, 86912, dtype, off)
    check(KERNELS[kernel], 4, 86912, dtype, weight_off=2)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,M,N", [("bf16", 3, 81984), ("fp16", 2, 90113), ("fp32", 3, 49156), ("fp16_res32", 60, 100003), WHOLE])
def test_a_captured_call_runs_the_kernel_tested_as_such(dtype, M, N):
    x, xok, r, rok, w = norm_inputs(M, N, dtype, N)
    x0, r0, xw, rw = x.clone(), r.clone(), x.clone(), r.clone()
    B.addrms_run(x, r, w, 1e-6, M, N, dtype)                      # prepares the kernel
    if (dtype, M, N) == WHOLE:
        xw, rw = x.clone(), r.clone()
    else:
        B.addrms_whole_rows_probe(xw, rw, w, 1e-6, M, N, dtype, True)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        B.addrms_run(x, r, w, 1e-6, M, N, dtype)
    for _ in range(3):
        x.copy_(x0)
        r.copy_(r0)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(bits(r), bits(rw)) and torch.equal(bits(x), bits(xw)) and xok() and rok()
