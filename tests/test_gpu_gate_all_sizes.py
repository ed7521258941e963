"""Comparisons of more workgroups than one, in one launch: the last workgroup folds the counts of all others.  Around the most
workgroups that a launch has, around the lanes of the folding one, and more launches at once than there are units for."""
import pytest
import torch

from paper_2601_12698_amd import binding as B
from test_zz_no_alloc import counts, planted

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "fp16_res32", "fp32"])
@pytest.mark.parametrize("workgroups,more", [(64, 1), (65, 0), (97, 3), (511, 0), (511, 1), (512, 0), (512, 5), (1024, 1)])
def test_counts(dtype, workgroups, more):
    n = workgroups * 512 * (4 if dtype == "fp32" else 8) + more
    case = planted(dtype, n, n, 7, 11, 2)
    for tol in (0, 1):
        assert counts(B.addrms_gate_probe_noalloc, case, dtype, tol) == counts(B.addrms_gate_probe, case, dtype, tol)


@pytest.mark.parametrize("looks", [0, 1, 1000])
@pytest.mark.parametrize("dtype,n", [("bf16", 4097), ("fp16_res32", 64 * 4096), ("fp32", 65 * 2048 + 3), ("bf16", 512 * 4096 + 9)])
def test_workgroups_that_are_not_there(dtype, n, looks):
    """The one that adds up compares the elements of those whose counts it does not find."""
    case = planted(dtype, n, 3, 40, 11, 2)
    for tol in (0, 1):
        want = counts(B.addrms_gate_probe, case, dtype, tol)
        assert counts(lambda y, v, r, q, d, t, o: B.addrms_gate_looks_probe(y, v, r, q, d, t, looks, o), case, dtype, tol) == want


def test_units_come_back():
    """More comparisons than there are units, each over before the next: one whose end is lost would leave too few of them."""
    case, out = planted("bf16", 20000, 1, 3, 5, 2), torch.zeros(4, dtype=torch.int32, device="cuda")
    for _ in range(600):
        B.addrms_gate_looks_probe(*case, "bf16", 1, 1000, out)
        torch.cuda.synchronize()


def test_more_launches_than_units():
    """600 launches in flight, of sizes in turn, so that every unit is used again with words of another launch in it."""
    per = 512 * 8
    cases = [planted("bf16", n, n, 3, 5, 2) for n in (2 * per, 40 * per + 1, 300 * per, 3 * per, 512 * per)]
    want = [counts(B.addrms_gate_probe, c, "bf16", 1) for c in cases]
    outs = [torch.full((4,), -1, dtype=torch.int32, device="cuda") for _ in range(600)]
    torch.cuda.synchronize()
    for i, o in enumerate(outs):
        B.addrms_gate_probe_noalloc(*cases[i % 5], "bf16", 1, o)
    torch.cuda.synchronize()
    got = [tuple(int(v) & 0xffffffff for v in o.cpu().tolist()) for o in outs]
    assert got == [want[i % 5] for i in range(600)]
