"""A *_run call keeps what it decided for a problem (kernel, launch shape, checks passed) and decides anew when anything
it depends on differs: the sizes, the format, the configuration, the table, the alignment of the tensors."""
import threading

import pytest
import torch

from paper_2601_12698_amd import binding as B
from test_gpu_untuned import bits, norm_inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _empty_table():
    B.addrms_table_clear()
    yield
    B.addrms_table_clear()


def run_and_check(M, N, dtype, off=0, cfg=None, seed=0):
    x, xok, r, rok, w = norm_inputs(M, N, dtype, seed, off)
    xw, rw, ww = x.clone(), r.clone(), w.clone()
    ref = B.make_cfg(1, 256, 1)                                    # one element per access: no alignment to speak of
    B.addrms_run(xw, rw, ww, 1e-6, M, N, dtype, ref)
    B.addrms_run(x, r, w, 1e-6, M, N, dtype, cfg)
    torch.cuda.synchronize()
    assert torch.equal(bits(x), bits(xw)) and torch.equal(bits(r), bits(rw)) and xok() and rok()


def test_the_table_decides_from_its_next_change_on():
    M, N = 9, 1000
    for _ in range(2):
        run_and_check(M, N, "bf16")
        with pytest.raises(B.AddrmsError) as e:
            run_and_check(M, N, "bf16", off=1)                     # the default configuration reads 16 bytes at a time
        assert e.value.status == B.ERR_MISALIGNED
        B.addrms_table_insert(M, N, "bf16", B.make_cfg(1, 256, 1))
        run_and_check(M, N, "bf16", off=1)
        run_and_check(M, N, "bf16")
        B.addrms_table_clear()


def test_alignment_is_looked_at_in_every_call():
    M, N, cfg = 9, 1000, B.make_cfg(8, 128, 1)
    for off in (0, 1, 0, 4, 8, 0):
        if off * 2 % 16 == 0:
            run_and_check(M, N, "bf16", off, cfg)
            continue
        with pytest.raises(B.AddrmsError) as e:
            run_and_check(M, N, "bf16", off, cfg)
        assert e.value.status == B.ERR_MISALIGNED


def test_calls_that_differ_in_one_thing_only():
    """More of them than a thread keeps, twice over, so that later ones push earlier ones out."""
    for rep in range(2):
        for N in range(512, 512 + 24 * 4, 4):
            for M in (3, 4):
                for dtype in ("bf16", "fp16"):
                    run_and_check(M, N, dtype, seed=rep + N)
                run_and_check(M, N, "bf16", cfg=B.make_cfg(4, 128, 1, flags=B.FLAG_NONTEMPORAL))
    bad = B.make_cfg(8, 128, 16)
    x, _, r, _, w = norm_inputs(3, 1000, "bf16", 0)
    for _ in range(2):                                             # refused every time, not only the first
        with pytest.raises(B.AddrmsError) as e:
            B.addrms_run(x, r, w, 1e-6, 3, 1000, "bf16", bad)
        assert e.value.status == B.ERR_INFEASIBLE_CFG and B.addrms_last_error()


def test_threads_on_streams_of_their_own():
    failures = []

    def work(k):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for i in range(20):
                    run_and_check(5 + k, 768 + 8 * (i % 3), "bf16", seed=100 * k + i)
        except Exception as e:                                     # noqa: BLE001
            failures.append(repr(e))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not failures, failures
