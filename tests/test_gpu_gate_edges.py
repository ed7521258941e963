"""The gate takes 16 bytes of a tensor per access: lengths around a whole number of pieces and of workgroups, and
tensors that start at any element."""
import numpy as np
import pytest
import torch

from paper_2601_12698_amd import binding as B
from test_gpu_gate import R_T, X_T, int_view, run_gate

pytestmark = pytest.mark.gpu


def expected(y, y_ref, r, r_ref, tol):
    def ordered(t):
        v = int_view(t).cpu().numpy().astype(np.int64)
        return np.where(v < 0, -(v + (1 << (8 * t.element_size() - 1))), v)
    d = np.abs(ordered(y) - ordered(y_ref))
    rbad = int((int_view(r).cpu() != int_view(r_ref).cpu()).sum())
    return rbad, int((d > tol).sum()), int(d.max())


@pytest.mark.parametrize("dtype", ["bf16", "fp16", "fp16_res32", "fp32"])
@pytest.mark.parametrize("n", [2, 3, 4, 5, 7, 8, 9, 15, 17, 2047, 2049, 4095, 4103, 8191, 524_288 * 8 + 5])
def test_gate_counts_any_length_and_start(dtype, n):
    """Random bit patterns of either sign, most elements wrong; exact counts, so no tolerance."""
    g = torch.Generator().manual_seed(n)
    bits = lambda t, m: torch.randint(-(1 << (8 * t.itemsize - 1)), 1 << (8 * t.itemsize - 1), (m,), generator=g)
    for off in (0, 1, 3):
        def make(t):
            iv = torch.int16 if t.itemsize == 2 else torch.int32
            return bits(t, n + off).to(iv).cuda().view(t)[off:]
        y, y_ref, r, r_ref = make(X_T[dtype]), make(X_T[dtype]), make(R_T[dtype]), make(R_T[dtype])
        int_view(r)[: n // 2] = int_view(r_ref)[: n // 2]
        int_view(y)[: n // 3] = int_view(y_ref)[: n // 3]
        for tol in (0, 1000):
            assert run_gate(y, y_ref, r, r_ref, dtype, tol) == expected(y, y_ref, r, r_ref, tol), (dtype, n, off, tol)
