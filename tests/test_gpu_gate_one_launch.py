"""Small comparisons are one launch whose last workgroup folds the counts of all: on either side of one workgroup and of the
most that meet, call after call, and recorded in a graph (where they are two launches)."""
import ctypes
import os

import pytest
import torch

from paper_2601_12698_amd import binding as B
from test_zz_no_alloc import R_T, X_T, counts, planted

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "fp16_res32", "fp32"])
def test_same_counts_as_two_launches(dtype):
    per = 512 * (4 if dtype == "fp32" else 8)                     # elements of a workgroup
    sizes = (per, per + 1, 2 * per, 2 * per + 1, 95 * per, 96 * per, 96 * per + 1, 7)
    cases = [planted(dtype, n, n, min(3, n // 2), min(5, n // 3), min(2, n // 4)) for n in sizes]
    want = [[counts(B.addrms_gate_probe, c, dtype, tol) for c in cases] for tol in (0, 1)]
    outs = []
    for _ in range(3):                                            # enqueued without a wait between them, large and small in turn
        for tol in (0, 1):
            for c in cases:
                outs.append(torch.full((4,), -1, dtype=torch.int32, device="cuda"))
                B.addrms_gate_probe_noalloc(*c, dtype, tol, outs[-1])
    torch.cuda.synchronize()
    got = [tuple(int(v) & 0xffffffff for v in o.cpu().tolist()) for o in outs]
    assert got == 3 * (want[0] + want[1])


def test_everything_wrong_in_as_many_elements_as_meet():
    n = 96 * 4096
    y = torch.zeros(n, dtype=X_T["bf16"], device="cuda")
    r = torch.zeros(n, dtype=R_T["bf16"], device="cuda")
    args = (y, (y.view(torch.int16) + 0x7f7f).view(y.dtype), r, (r.view(torch.int16) + 1).view(r.dtype))
    assert counts(B.addrms_gate_probe_noalloc, args, "bf16", 1) == (n, n, 0x7f7f, 0)
    y32 = torch.zeros(4097, dtype=torch.float32, device="cuda")
    far = torch.full_like(y32, float("nan")).view(torch.int32)
    far[:] = -1                                                   # the largest distance a format has
    assert counts(B.addrms_gate_probe_noalloc, (y32, far.view(torch.float32), y32, y32), "fp32", 1) == (0, 4097, 0x7fffffff, 0)


def test_streams_of_their_own_and_a_graph():
    cases = [planted("bf16", 5000 * (k + 1), k, 3 + k, 4, 5) for k in range(6)]
    want = [counts(B.addrms_gate_probe, c, "bf16", 1) for c in cases]
    outs = [torch.zeros(4, dtype=torch.int32, device="cuda") for _ in cases]
    torch.cuda.synchronize()
    for c, o in zip(cases, outs):
        s = torch.cuda.Stream()
        B.addrms_gate_probe_noalloc(*c, "bf16", 1, o, s)
        s.synchronize()
    assert [tuple(o.cpu().tolist()) for o in outs] == want
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        for c, o in zip(cases, outs):
            B.addrms_gate_probe_noalloc(*c, "bf16", 1, o)
    for _ in range(3):
        for o in outs:
            o.fill_(-1)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert [tuple(o.cpu().tolist()) for o in outs] == want
        assert counts(B.addrms_gate_probe_noalloc, cases[3], "bf16", 1) == want[3]


def test_an_older_error_of_the_callers_is_not_the_launchs():
    """A call that failed before, an invalid device asked for, leaves its error pending in the thread: the comparison is
    queued all the same, and says so, and the error stays for whoever asks for it."""
    case = planted("bf16", 5000, 3, 3, 4, 5)
    want = counts(B.addrms_gate_probe, case, "bf16", 1)
    out = torch.zeros(4, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    hip = ctypes.CDLL(os.path.join(os.path.dirname(torch.__file__), "lib", "libamdhip64.so"))
    error = hip.hipSetDevice(9999)
    assert error != 0
    try:
        B.addrms_gate_probe_noalloc(*case, "bf16", 1, out)
        pending = hip.hipPeekAtLastError()
    finally:
        hip.hipGetLastError()
    torch.cuda.synchronize()
    assert pending == error and tuple(out.cpu().tolist()) == want
