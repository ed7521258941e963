"""Which kernel a call without a configuration takes (the rules are host code): that every kernel built can be asked for
and none is asked for that does not exist, that launch shapes cover their rows, what each side of each limit takes, and
that the cases of the GPU tests run the kernels they are meant for."""
import os
import shutil
import subprocess

import pytest

from paper_2601_12698_amd import binding as B
from test_gpu_untuned import LONG, MERGE, NORM, RAGGED, SILU
from test_host_sanitizers import BUILD, CSRC, HOST_SOURCES, ROOT


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    if not os.path.exists(os.path.join(BUILD, "gen_resources.inc")):
        pytest.skip("the generated instance and resource tables are not present (build the library first)")
    exe = str(tmp_path_factory.mktemp("route") / "driver")
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined", "-Wall", "-Wextra",
           "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-I", BUILD, os.path.join(ROOT, "tests", "untuned_route_driver.cpp"),
           *[os.path.join(CSRC, s) for s in HOST_SOURCES + ["direct_route.cpp"]], "-o", exe]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=600)
    assert r.returncode == 0, r.stdout[-4000:]
    return exe


def routes(driver, problems):
    """(op, dtype, M, N[, x, r, w]) -> what the rules say, x, r, w being bytes past a multiple of 16."""
    lines = "\n".join(" ".join(map(str, (p[0], B.DTYPE_IDS[p[1]], *p[2:], *([0] * (7 - len(p)))))) for p in problems)
    r = subprocess.run([driver], input=lines, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=120)
    assert r.returncode == 0, r.stdout[-4000:]
    out = r.stdout.split("\n")[:-1]
    assert len(out) == len(problems), r.stdout[-4000:]
    return out


def test_the_kernels_asked_for_are_the_kernels_built(driver):
    r = subprocess.run([driver, "walk"], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-4000:]


def test_the_gpu_cases_run_what_they_are_meant_for(driver):
    for (dtype, M, N), got in zip(NORM, routes(driver, [("addrms", *c) for c in NORM])):
        assert got.startswith("row") and "ragged" not in got, (dtype, M, N, got)
    # on the other side of a limit: too small; one element longer than the registers
    beside = {("bf16", 67, 129): "default", ("bf16", 66, 131): "default", ("fp16", 130, 255): "default", ("bf16", 5, 450): "default", ("bf16", 40, 1030): "default", ("fp16", 2, 32707): "long cached ragged parked=0",
              ("fp32", 2, 32739): "long cached ragged parked=0"}
    for (dtype, M, N), got in zip(RAGGED, routes(driver, [("addrms", *c) for c in RAGGED])):
        want = beside.get((dtype, M, N))
        assert got == want if want else got.startswith("row") and "ragged" in got, (dtype, M, N, got)
    for (dtype, M, N), got in zip(LONG, routes(driver, [("addrms", *c) for c in LONG])):
        assert got.startswith("long"), (dtype, M, N, got)
    for (dtype, M, d), got in zip(SILU, routes(driver, [("silumul", *c) for c in SILU])):
        vec = 4 if dtype == "fp32" else 8
        want = got == "default" if d < 2 * vec else got.startswith("flat") and ("ragged" in got) == (d % vec != 0)
        assert want, (dtype, M, d, got)
    for (dtype, rows, d), got in zip(MERGE, routes(driver, [("merge", *c) for c in MERGE])):
        assert (got == "default") == (d % 8 != 0 or rows * d * 6 < 4 << 20), (dtype, rows, d, got)
    assert routes(driver, [("merge", "bf16", 11 * 700, 128), ("merge", "fp16", 7 * 500, 256)]) == ["flat writethrough"] * 2


LIMITS = [
    # rows shorter than sixteen accesses; the longest row of the registers
    (("addrms", "bf16", 64, 120), "default"),
    (("addrms", "bf16", 64, 128), "row nontemporal pieces=1 threads=32 rows=2"),
    (("addrms", "bf16", 8, 32768), "row writethrough pieces=4 threads=1024 rows=1"),
    (("addrms", "bf16", 8, 32832), "long cached parked=0"),
    # store policy: 512 KB and 96 MB of x and residual
    (("addrms", "bf16", 127, 1024), "row nontemporal pieces=1 threads=128 rows=1"),
    (("addrms", "bf16", 128, 1024), "row writethrough pieces=1 threads=128 rows=1"),
    (("addrms", "bf16", 6144, 4096), "row writethrough pieces=2 threads=256 rows=1"),
    (("addrms", "bf16", 6145, 4096), "row nontemporal pieces=1 threads=512 rows=1"),
    (("addrms", "bf16", 614, 40960), "long cached parked=0"),
    (("addrms", "bf16", 615, 40960), "long nontemporal parked=0"),
    # whole vectors but not whole lines: ordinary loads from 512 KB on; walked by lines from 16 MB and 64 pieces on, and then
    # only rows of up to 3 KB of x; never non-temporal loads where waves share lines
    (("addrms", "bf16", 131, 1000), "row nontemporal pieces=1 threads=128 rows=1"),
    (("addrms", "bf16", 132, 1000), "row shared pieces=1 threads=128 rows=1"),
    (("addrms", "fp16", 139, 30008), "row shared pieces=4 threads=960 rows=1"),
    (("addrms", "fp16", 140, 30008), "row writethrough ragged pieces=4 threads=960 rows=1"),
    (("addrms", "bf16", 30000, 504), "row shared pieces=1 threads=64 rows=1"),
    (("addrms", "bf16", 30000, 520), "row shared ragged pieces=2 threads=64 rows=2"),
    (("addrms", "bf16", 9000, 1528), "row shared ragged pieces=2 threads=128 rows=2"),
    (("addrms", "bf16", 9000, 1544), "row writethrough ragged pieces=2 threads=128 rows=2"),
    (("addrms", "bf16", 228658, 328), "row shared pieces=1 threads=64 rows=1"),
    (("addrms", "fp32", 500000, 100), "row shared pieces=1 threads=32 rows=2"),
    (("addrms", "bf16", 62500, 1000), "row shared ragged pieces=1 threads=192 rows=1"),
    (("addrms", "bf16", 62500, 2056), "row nontemporal ragged pieces=1 threads=320 rows=1"),
    (("silumul", "bf16", 4096, 12288), "flat writethrough"),
    (("silumul", "bf16", 4097, 12288), "flat nontemporal"),
    (("merge", "bf16", 196608, 256), "flat writethrough"),
    (("merge", "bf16", 196609, 256), "flat nontemporal"),
    (("merge", "bf16", 2709, 256), "default"),
    (("merge", "bf16", 2710, 256), "flat writethrough"),
    # single elements: small ones are the default configuration's, up to 1 to 2 MB where its accesses are wide or rows short
    (("addrms", "bf16", 254, 1030), "default"),
    (("addrms", "bf16", 255, 1030), "row nontemporal ragged pieces=1 threads=192 rows=1"),
    (("addrms", "bf16", 562, 932), "default"),
    (("addrms", "bf16", 563, 932), "row nontemporal ragged pieces=1 threads=128 rows=2"),
    (("addrms", "bf16", 765, 514), "default"),
    (("addrms", "bf16", 766, 514), "row nontemporal ragged pieces=1 threads=128 rows=2"),
    (("addrms", "bf16", 2031, 129), "default"),
    (("addrms", "bf16", 2033, 129), "row nontemporal ragged pieces=1 threads=32 rows=2"),
    (("addrms", "bf16", 5, 259), "row nontemporal ragged pieces=1 threads=64 rows=1"),
    (("addrms", "fp32", 130, 1002), "default"),
    (("addrms", "fp32", 131, 1002), "row nontemporal ragged pieces=1 threads=320 rows=1"),
    (("addrms", "fp32", 5, 65), "row nontemporal ragged pieces=1 threads=32 rows=2"),
    # three pieces per thread from 4 MB, two rows per workgroup; one piece beyond 96 MB; never write-through
    (("addrms", "bf16", 1047, 1001), "row nontemporal ragged pieces=1 threads=192 rows=2"),
    (("addrms", "bf16", 1048, 1001), "row nontemporal ragged pieces=3 threads=64 rows=2"),
    (("addrms", "bf16", 511, 2055), "row nontemporal ragged pieces=3 threads=128 rows=1"),
    (("addrms", "fp16", 2047, 4095), "row nontemporal ragged pieces=3 threads=192 rows=2"),
    (("addrms", "bf16", 9000, 6150), "row nontemporal ragged pieces=1 threads=832 rows=1"),
    # bases: the streams at different elements, the weights alone off a 16-byte address, a base no access fits
    (("addrms", "bf16", 17, 1001, 2, 2, 2), "row nontemporal ragged pieces=1 threads=192 rows=1"),
    (("addrms", "bf16", 17, 1001, 2, 0, 2), "default"),
    (("addrms", "bf16", 17, 1000, 2, 2, 2), "misaligned"),
    (("silumul", "bf16", 9, 1001, 2, 0), "flat writethrough ragged"),
    (("silumul", "bf16", 9, 1001, 2, 2), "default"),
    # what the default configuration refuses stays refused
    (("silumul", "bf16", 2, 8193), "refused"),
    (("addrms", "bf16", 1, (1 << 28) + 8), "refused"),
]


def test_both_sides_of_each_limit(driver):
    got = routes(driver, [p for p, _ in LIMITS])
    assert [(p, g) for (p, _), g in zip(LIMITS, got)] == LIMITS


def test_launches_of_more_threads_than_fit_are_left_to_the_default(driver):
    assert routes(driver, [("addrms", "bf16", 2 ** 27 - 2, 128), ("addrms", "bf16", 2 ** 27, 128), ("silumul", "bf16", 2 ** 20, 2047),
                           ("silumul", "bf16", 2 ** 20, 2048), ("merge", "bf16", 2 ** 23 - 1, 256), ("merge", "bf16", 2 ** 23, 256)]) == \
        ["row nontemporal pieces=1 threads=32 rows=2", "default", "flat nontemporal ragged", "default", "flat nontemporal", "default"]
