"""Ragged rows, which share cache lines with the row before and behind: ordinary loads or non-temporal ones, of their single elements
in add+RMSNorm and of all in silu_and_mul (host code, on the CPU), and rows that are read either way (on the GPU)."""
import subprocess

import pytest

from paper_2601_12698_amd import binding as B
from test_few_rows import driver                            # noqa: F401
from test_gpu_untuned import check_norm

# both sides of each limit: rows of 3 KB of x; 16, 36 and 64 MB of x and residual; rows of 16000 bytes of x
CASES = [
    (("fp16", 5000, 1535), "ordinary"), (("fp16", 5000, 1537), "nontemporal"), (("fp16", 2700, 1537), "ordinary"),
    (("bf16", 1048, 4001), "ordinary"), (("bf16", 1049, 4001), "nontemporal"), (("bf16", 2358, 4001), "nontemporal"), (("bf16", 2359, 4001), "ordinary"),
    (("fp32", 2400, 767), "ordinary"), (("fp32", 2740, 769), "nontemporal"), (("fp32", 1179, 3999), "nontemporal"), (("fp32", 1180, 3999), "ordinary"),
    (("fp32", 1180, 4001), "nontemporal"), (("fp32", 2096, 4001), "nontemporal"), (("fp32", 2097, 4001), "ordinary"),
    (("fp16_res32", 1400, 2001), "nontemporal"), (("fp16_res32", 1400, 1501), "ordinary"), (("fp16", 64, 4096), "none"),
]


def test_both_sides_of_each_limit(driver):                  # noqa: F811
    lines = "\n".join(f"{B.DTYPE_IDS[d]} {M} {N}" for (d, M, N), _ in CASES)
    r = subprocess.run([driver, "singles"], input=lines, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=120)
    assert r.returncode == 0, r.stdout[-4000:]
    assert [(p, g) for (p, _), g in zip(CASES, r.stdout.split("\n"))] == CASES


# 26 MB of output
SILU = [(("bf16", 3325, 4099), "ordinary"), (("bf16", 3326, 4099), "nontemporal"), (("fp32", 6662, 1023), "ordinary"), (("fp32", 6663, 1023), "nontemporal"),
        (("fp16", 1, 8191), "ordinary"), (("bf16", 3325, 4096), "none")]


def test_both_sides_of_the_limit_of_activations(driver):    # noqa: F811
    lines = "\n".join(f"{B.DTYPE_IDS[d]} {M} {N}" for (d, M, N), _ in SILU)
    r = subprocess.run([driver, "singles", "silu"], input=lines, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=120)
    assert r.returncode == 0, r.stdout[-4000:]
    assert [(p, g) for (p, _), g in zip(SILU, r.stdout.split("\n"))] == SILU


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,M,N", [c for c, how in CASES if how != "none"])
def test_rows(dtype, M, N):
    B.addrms_table_clear()
    check_norm(M, N, dtype)
