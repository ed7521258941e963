"""Rows that are split over several workgroups: who may use which units of the memory they meet in, and the shapes in which
rows are split (host code, on the CPU); the kernel itself, with every wait cut short, beside other streams and beyond the
rows of one launch (on the GPU)."""
import os
import re
import shutil
import subprocess

import pytest
import torch

from paper_2601_12698_amd import binding as B
from paper_2601_12698_amd import build
from test_gpu_untuned import bits, check_norm, norm_inputs
from test_host_sanitizers import BUILD, CSRC, HOST_SOURCES, ROOT


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    if not os.path.exists(os.path.join(BUILD, "gen_resources.inc")):
        pytest.skip("the generated instance and resource tables are not present (build the library first)")
    exe = str(tmp_path_factory.mktemp("split") / "driver")
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined", "-Wall", "-Wextra",
           "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-I", BUILD, os.path.join(ROOT, "tests", "split_rows_driver.cpp"),
           *[os.path.join(CSRC, s) for s in HOST_SOURCES + ["direct_route.cpp"]], "-o", exe]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=600)
    assert r.returncode == 0, r.stdout[-4000:]
    return exe


@pytest.mark.parametrize("what", ["slots", "walk"])
def test_slots_and_shapes(driver, what):
    r = subprocess.run([driver, what], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-4000:]


def test_registers_leave_room_for_workgroups():
    """Waves per SIMD of the kernels with four pieces per thread: what the sizes of the parts were measured with.  A CU holds two
    workgroups of 1024 threads, and three of 384 (16-bit rows), 512 where they are ragged."""
    path = os.path.join(BUILD, "addrms_split.remarks")
    if not os.path.exists(path):
        pytest.skip("the library is not built here")
    seen = 0
    with open(path) as f:
        kernels = build.parse_remarks(f.read())
    for name, r in kernels.items():
        m = re.search(r"addrms_splitILi(\d)ELi(\d)ELi(\d)ELi(\d)ELb(\d)E", name)
        if m:
            seen += 1
            _, vec, pieces, _, ragged = map(int, m.groups())
            least = 8 if pieces < 4 or vec == 4 else 6 if ragged else 5
            assert r["occupancy"] >= least and r["scratch"] == 0, (name, r)
    assert seen == 32


def test_parts_of_whole_16_bit_rows_are_two_to_a_cu():
    """Five waves per SIMD, no more: two workgroups of 512 threads, which is faster than three."""
    path = os.path.join(BUILD, "addrms_split.remarks")
    if not os.path.exists(path):
        pytest.skip("the library is not built here")
    with open(path) as f:
        waves = [r["occupancy"] for name, r in build.parse_remarks(f.read()).items() if re.search(r"addrms_splitILi\dELi8ELi4ELi\dELb0E", name)]
    assert waves and set(waves) == {5}


SHAPES = [
    (("bf16", 8, 32832), "parts=9 threads=512 pieces=1 nontemporal"),
    (("bf16", 1024, 131072), "parts=8 threads=512 pieces=4 nontemporal"),
    (("fp32", 500, 200000), "parts=16 threads=832 pieces=4 nontemporal"),
    (("bf16", 1, 200000), "parts=16 threads=832 pieces=2 nontemporal"),
    (("fp16", 46, 164992), "parts=11 threads=960 pieces=2 nontemporal"),
    # write-through from 32 MB to 96 MB of x and residual
    (("bf16", 64, 131072), "parts=8 threads=1024 pieces=2 nontemporal"),
    (("bf16", 69, 121344), "parts=8 threads=512 pieces=4 nontemporal"),
    (("bf16", 70, 121344), "parts=8 threads=512 pieces=4 writethrough"),
    (("bf16", 207, 121344), "parts=8 threads=512 pieces=4 writethrough"),
    (("bf16", 208, 121344), "parts=8 threads=512 pieces=4 nontemporal"),
    # rows that one workgroup holds, in numbers that fill the chip
    (("bf16", 159, 40960), "parts=3 threads=896 pieces=2 nontemporal"),
    (("bf16", 160, 40960), "whole"),
    (("bf16", 256, 40960), "whole"),
    (("bf16", 257, 40960), "parts=3 threads=448 pieces=4 writethrough"),
    (("bf16", 512, 40960), "whole"),
    (("bf16", 513, 40960), "parts=3 threads=448 pieces=4 writethrough"),
    (("bf16", 447, 57344), "parts=4 threads=448 pieces=4 nontemporal"),
    (("fp16_res32", 447, 32832), "parts=3 threads=704 pieces=4 writethrough"),
    (("fp16_res32", 448, 32832), "whole"),
    # 16-bit rows that its registers hold, where the last turn of the 256 CUs is not too empty: two, three or four
    # turns by their length
    (("bf16", 332, 40960), "parts=3 threads=448 pieces=4 writethrough"),
    (("bf16", 333, 40960), "whole"),
    (("bf16", 333, 49152), "whole"),
    (("bf16", 333, 49160), "parts=4 threads=448 pieces=4 writethrough"),
    (("bf16", 537, 40960), "parts=3 threads=448 pieces=4 writethrough"),
    (("bf16", 538, 40960), "whole"),
    (("bf16", 538, 41024), "parts=3 threads=448 pieces=4 writethrough"),
    (("bf16", 768, 40960), "whole"),
    (("bf16", 769, 40960), "parts=3 threads=448 pieces=4 nontemporal"),
    (("fp16", 769, 36864), "whole"),
    (("fp16", 769, 36928), "parts=3 threads=448 pieces=4 nontemporal"),
    (("fp16", 1024, 36864), "whole"),
    (("fp16", 1025, 36864), "parts=3 threads=384 pieces=4 nontemporal"),
    (("bf16", 600, 33333), "parts=3 threads=384 pieces=4 writethrough"),
    (("bf16", 200, 81920), "whole"),
    (("bf16", 200, 81984), "parts=6 threads=448 pieces=4 writethrough"),
    # the longest row, and one piece more
    (("bf16", 2, 524288), "parts=16 threads=1024 pieces=4 nontemporal"),
    (("bf16", 2, 524352), "whole"),
    (("fp32", 2, 262144), "parts=16 threads=1024 pieces=4 nontemporal"),
    (("fp32", 2, 262176), "whole"),
    (("bf16", 8, 32768), "whole"),
]


def test_both_sides_of_each_limit(driver):
    lines = "\n".join(f"{B.DTYPE_IDS[d]} {M} {N}" for (d, M, N), _ in SHAPES)
    r = subprocess.run([driver], input=lines, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=120)
    assert r.returncode == 0, r.stdout[-4000:]
    assert [(p, g) for (p, _), g in zip(SHAPES, r.stdout.split("\n"))] == SHAPES


# two parts and the most; last parts of one line and whole ones; one, two and four pieces per thread; ragged rows; both store
# policies
SPLIT = [("bf16", 2, 32832), ("bf16", 1300, 40960), ("fp16", 3, 32707), ("bf16", 1, 524288), ("fp16", 2, 262143), ("bf16", 70, 121344),
         ("fp32", 2, 32772), ("fp32", 1, 262144), ("fp32", 60, 131071), ("fp16_res32", 40, 40004), ("fp16_res32", 90, 86022), ("bf16", 33, 131008)]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,M,N", SPLIT)
def test_split_rows_give_the_bits_of_whole_ones(dtype, M, N):
    B.addrms_table_clear()
    check_norm(M, N, dtype)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,M,N", SPLIT)
@pytest.mark.parametrize("patience", [0, 2])
def test_sums_formed_in_place_of_others(dtype, M, N, patience):
    """As if the other workgroups of a row were not on the chip: whoever misses a sum forms it."""
    x, xok, r, rok, w = norm_inputs(M, N, dtype, N)
    xw, rw = x.clone(), r.clone()
    B.addrms_run(xw, rw, w, 1e-6, M, N, dtype, B.addrms_default_cfg(N, dtype))
    B.addrms_split_probe(x, r, w, 1e-6, M, N, dtype, patience)
    torch.cuda.synchronize()
    assert torch.equal(bits(r), bits(rw)) and torch.equal(bits(x), bits(xw)) and xok() and rok()


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,M,N", SPLIT)
def test_rows_of_calls_that_find_no_units(dtype, M, N):
    x, xok, r, rok, w = norm_inputs(M, N, dtype, N, special=[(0, 5, float("inf")), (M - 1, N - 1, float("nan"))] if M > 2 else None)
    xw, rw = x.clone(), r.clone()
    B.addrms_split_probe(xw, rw, w, 1e-6, M, N, dtype, 256)
    B.addrms_whole_rows_probe(x, r, w, 1e-6, M, N, dtype, False)
    torch.cuda.synchronize()
    assert torch.equal(bits(r), bits(rw)) and torch.equal(bits(x), bits(xw)) and xok() and rok()


# A row of 4096 elements b and then 2^-26 b, whose squares are lost one by one in a thread's sum that holds four b^2, but not
# where a part of the row has none of the b: the sums are 15 * 2^-50 apart, and rstd's fp32 rounding changes between them.
IN_BETWEEN = [float.fromhex(h) for h in ("0x1.457afap-6", "0x1.3e3ca4p-3", "0x1.738498p-3", "0x1.5bf846p-2", "0x1.0c41ep-1")]


@pytest.mark.gpu
def test_the_order_of_the_sum_does_not_depend_on_what_is_in_flight():
    """Bits of rows for which the order of the row sum decides: the same from split rows, where every sum is formed by others,
    and where no units are found.  (The kernel of captured calls adds in another order, which shows that the rows can tell.)"""
    M, N = len(IN_BETWEEN), 262144
    b = torch.tensor(IN_BETWEEN, dtype=torch.float64)[:, None].expand(M, N).clone()
    b[:, 4096:] *= 2.0 ** -26
    b[:, -1] = 2.0 ** -60                                         # its y is rstd, scaled
    x0, w = b.float().cuda(), torch.ones(N, device="cuda")
    assert torch.equal(x0.cpu().double(), b)
    outs = []
    for run in (lambda *a: B.addrms_run(*a), lambda *a: B.addrms_split_probe(*a, 0), lambda *a: B.addrms_whole_rows_probe(*a, False),
                lambda *a: B.addrms_whole_rows_probe(*a, True)):
        x, r = x0.clone(), torch.zeros_like(x0)
        run(x, r, w, 1e-6, M, N, "fp32")
        torch.cuda.synchronize()
        outs.append(bits(x))
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
    assert bool((outs[0][:, -1] != outs[3][:, -1]).all())


@pytest.mark.gpu
def test_problems_that_are_not_split_are_refused():
    x, _, r, _, w = norm_inputs(2, 4096, "bf16", 1)
    with pytest.raises(B.AddrmsError) as e:
        B.addrms_split_probe(x, r, w, 1e-6, 2, 4096, "bf16", 8)
    assert e.value.status == B.ERR_UNSUPPORTED_SHAPE


@pytest.mark.gpu
def test_more_rows_than_one_launch_takes():
    B.addrms_table_clear()
    check_norm(4099, 33000, "bf16")


@pytest.mark.gpu
def test_more_streams_than_slots():
    """Six streams with several launches in flight each."""
    B.addrms_table_clear()
    M, N, dtype = 300, 50000, "bf16"
    streams = [torch.cuda.Stream() for _ in range(6)]
    inputs = [norm_inputs(M, N, dtype, 11 * k) for k in range(6)]
    want = []
    for x, _, r, _, w in inputs:
        xw, rw = x.clone(), r.clone()
        for _ in range(5):
            B.addrms_run(xw, rw, w, 1e-6, M, N, dtype, B.addrms_default_cfg(N, dtype))
        want.append((xw, rw))
    torch.cuda.synchronize()
    for _ in range(5):
        for s, (x, _, r, _, w) in zip(streams, inputs):
            B.addrms_run(x, r, w, 1e-6, M, N, dtype, None, s)
    torch.cuda.synchronize()
    for (x, xok, r, rok, _), (xw, rw) in zip(inputs, want):
        assert torch.equal(bits(x), bits(xw)) and torch.equal(bits(r), bits(rw)) and xok() and rok()
    for _ in range(8):                                            # units are given back: a new stream can have some
        s = torch.cuda.Stream()
        x, _, r, _, w = inputs[0]
        B.addrms_split_probe(x, r, w, 1e-6, M, N, dtype, 256, s)
        s.synchronize()


@pytest.mark.gpu
def test_threads_that_launch_at_the_same_time():
    """Each on a stream of its own."""
    import threading
    B.addrms_table_clear()
    M, N, dtype, failures = 7, 40000, "bf16", []

    def work(k):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                x, xok, r, rok, w = norm_inputs(M, N, dtype, 3 * k)
                xw, rw = x.clone(), r.clone()
                for _ in range(30):
                    B.addrms_run(x, r, w, 1e-6, M, N, dtype)
                    B.addrms_run(xw, rw, w, 1e-6, M, N, dtype, B.addrms_default_cfg(N, dtype))
                torch.cuda.current_stream().synchronize()
                assert torch.equal(bits(x), bits(xw)) and torch.equal(bits(r), bits(rw)) and xok() and rok()
        except Exception as e:                                    # noqa: BLE001
            failures.append(repr(e))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(6)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not failures, failures
