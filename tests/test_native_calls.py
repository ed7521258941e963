"""The native form of the hot calls (module _native) against the general one: it takes the usual calls and nothing else, and
what it takes gives the same outputs, statuses and errors."""
import ctypes
import importlib.machinery
import os

import numpy as np
import pytest
import torch

from paper_2601_12698_amd import binding as B
from test_gpu_untuned import bits, finite, norm_inputs


class SubTensor(torch.Tensor):
    pass


class SubCfg(B.Cfg):
    pass


def test_the_module_is_built_and_leaves_what_is_not_usual_to_the_general_way():
    B._torch()
    n = B._native
    assert n is not None
    x = torch.zeros(4, 64, dtype=torch.bfloat16)                  # not on a device: everything else is as it should be
    s = torch.zeros(4)
    assert n.addrms_run(x, x, x[0], 1e-6, 4, 64, "bf16", None) is None
    assert n.silumul_run(x, x, 2, 64, "bf16", None) is None
    assert n.mergestates_run(x, s, x, s, x, s, 4, 64, "bf16", None) is None
    assert n.addrms_gate_probe_noalloc(x, x, x, x, "bf16", 1, s) is None
    for args in ((), (1, 2, 3), (None,) * 8, (x, x, x[0], 1, 4, 64, "bf16", None), (x, x, x[0], 1e-6, 1 << 63, 64, "bf16", None),
                 (x, x, x[0], 1e-6, 1 << 62, 1 << 62, "bf16", None), (x, x, x[0], 1e-6, 4, 64, "int8", None),
                 (x, x, x[0], 1e-6, 4, 64, 4, None), (x, x, x[0], 1e-6, 4, 64, [], None), (x, x, x[0], 1e-6, 4, 64, "bf16", 5)):
        assert n.addrms_run(*args) is None
    with pytest.raises(TypeError):
        n.bind(B.DTYPE_IDS, B.Cfg)
    with pytest.raises(ValueError, match="device tensor"):
        B.addrms_run(x, x, x[0], 1e-6, 4, 64, "bf16")


def test_a_module_built_for_another_torch_is_not_used(monkeypatch):
    """It loads where the symbols it needs are there, but reads torch's objects where its own headers said."""
    B._torch()
    monkeypatch.setattr(B._native, "TORCH", "2.0.0 0000")
    monkeypatch.setattr(B, "_torch_facts", None)
    monkeypatch.setattr(B, "_native", None)
    B._torch()
    assert B._native is None
    monkeypatch.undo()
    assert B._native is not None and B._native.TORCH == B.torch_identity()


def test_a_build_without_torchs_headers_warns_and_goes_on(monkeypatch, tmp_path):
    """And a module for another torch or Python is built anew."""
    from paper_2601_12698_amd import build
    assert build.NATIVE.endswith(importlib.machinery.EXTENSION_SUFFIXES[0]) and os.path.exists(build.NATIVE)
    ran = []

    def run(cmd, **kw):
        ran.append(cmd[0])
        raise RuntimeError("no compiler")
    monkeypatch.setattr(build, "_run", run)
    build.build_native(force=False)                               # built already
    assert not ran
    monkeypatch.setattr(build, "NATIVE", str(tmp_path / "module.so"))
    (tmp_path / "module.so").write_bytes(b"built for some other torch")
    with pytest.warns(UserWarning, match="no compiler"):
        build.build_native(force=False)
    assert ran == ["g++"]


def outcome(monkeypatch, native, make, call):
    """What a call does: its outputs' bits, or its error."""
    state = make()
    with monkeypatch.context() as m:
        if not native:
            m.setattr(B, "_native", None)
        try:
            got = call(*state)
            torch.cuda.synchronize()
        except Exception as e:                                    # noqa: BLE001
            return type(e), str(e)
    assert got is None
    return [bits(t).cpu() for t in state]


def norm(M=9, N=1000, dtype="bf16"):
    x, _, r, _, w = norm_inputs(M, N, dtype, 5)
    return x, r, w


CALLS = {
    "plain": (norm, lambda x, r, w: B.addrms_run(x, r, w, 1e-6, 9, 1000, "bf16")),
    "format by number, keywords": (norm, lambda x, r, w: B.addrms_run(x, r, w, eps=1e-6, M=9, N=1000, dtype=0, cfg=None, stream=None)),
    "mixed formats": (lambda: norm(dtype="fp16_res32"), lambda x, r, w: B.addrms_run(x, r, w, 1e-6, 9, 1000, "fp16_res32")),
    "eps is an integer": (norm, lambda x, r, w: B.addrms_run(x, r, w, 1, 9, 1000, "bf16")),
    "a configuration": (norm, lambda x, r, w: B.addrms_run(x, r, w, 1e-6, 9, 1000, "bf16", B.make_cfg(4, 128, 2))),
    "a configuration's subclass": (norm, lambda x, r, w: B.addrms_run(x, r, w, 1e-6, 9, 1000, "bf16", SubCfg(4, 256, 1, 0, 1, 0, 0, 0))),
    "an infeasible configuration": (norm, lambda x, r, w: B.addrms_run(x, r, w, 1e-6, 9, 1000, "bf16", B.make_cfg(8, 128, 16))),
    "a bare number as configuration": (norm, lambda x, r, w: B.addrms_run(x, r, w, 1e-6, 9, 1000, "bf16", 7)),
    "other sizes than the tensors'": (norm, lambda x, r, w: B.addrms_run(x, r, w, 1e-6, 10, 1000, "bf16")),
    "another format than the tensors'": (norm, lambda x, r, w: B.addrms_run(x, r, w, 1e-6, 9, 1000, "fp16")),
    "no such format": (norm, lambda x, r, w: B.addrms_run(x, r, w, 1e-6, 9, 1000, "fp8")),
    "no such number of a format": (norm, lambda x, r, w: B.addrms_run(x, r, w, 1e-6, 9, 1000, -1)),
    "weights elsewhere": (norm, lambda x, r, w: B.addrms_run(x, r, w.cpu(), 1e-6, 9, 1000, "bf16")),
    "transposed": (norm, lambda x, r, w: B.addrms_run(x.view(9, 1000).t(), r, w, 1e-6, 9, 1000, "bf16")),
    "off its alignment": (norm, lambda x, r, w: B.addrms_run(x[1:-7], r[:-8], w[:-8], 1e-6, 1, 8992, "bf16")),
    "no rows": (norm, lambda x, r, w: B.addrms_run(x[:0], r[:0], w, 1e-6, 0, 1000, "bf16")),
    "a numpy integer": (norm, lambda x, r, w: B.addrms_run(x, r, w, 1e-6, np.int64(9), 1000, "bf16")),
    "a truth value": (lambda: norm(1), lambda x, r, w: B.addrms_run(x, r, w, 1e-6, True, 1000, "bf16")),
    "a parameter and a subclass": (norm, lambda x, r, w: B.addrms_run(x.as_subclass(SubTensor), r, torch.nn.Parameter(w), 1e-6, 9, 1000, "bf16")),
    "a stream": (norm, lambda x, r, w: B.addrms_run(x, r, w, 1e-6, 9, 1000, "bf16", None, torch.cuda.current_stream())),
    "not a tensor": (norm, lambda x, r, w: B.addrms_run(x, r, None, 1e-6, 9, 1000, "bf16")),
    "meta tensors": (norm, lambda x, r, w: B.addrms_run(x.to("meta"), r, w, 1e-6, 9, 1000, "bf16")),
    "activation": (lambda: (finite((7, 128), torch.float16, 1), torch.zeros(7, 64, device="cuda", dtype=torch.float16)),
                   lambda x, o: B.silumul_run(x, o, 7, 64, "fp16")),
    "activation, refused": (lambda: (finite((2, 16386), torch.bfloat16, 1), torch.zeros(2, 8193, device="cuda", dtype=torch.bfloat16)),
                            lambda x, o: B.silumul_run(x, o, 2, 8193, "bf16")),
    "activation, output too small": (lambda: (finite((7, 128), torch.float16, 1), torch.zeros(7, 63, device="cuda", dtype=torch.float16)),
                                     lambda x, o: B.silumul_run(x, o, 7, 64, "fp16")),
    "merge": (lambda: (*(finite((5, 64), torch.bfloat16, s) for s in (1, 2, 3)), *(finite((5,), torch.float32, s) for s in (4, 5, 6))),
              lambda a, b, o, sa, sb, so: B.mergestates_run(a, sa, b, sb, o, so, 5, 64, "bf16")),
    "merge, scores of another type": (lambda: (*(finite((5, 64), torch.bfloat16, s) for s in (1, 2, 3)), *(finite((5,), torch.float32, s) for s in (4, 5, 6))),
                                      lambda a, b, o, sa, sb, so: B.mergestates_run(a, sa.bfloat16(), b, sb, o, so, 5, 64, "bf16")),
    "gate": (lambda: (*(finite((5, 64), torch.bfloat16, s) for s in (1, 2, 3, 4)), torch.zeros(4, device="cuda", dtype=torch.int32)),
             lambda y, v, r, q, c: B.addrms_gate_probe_noalloc(y, v, r, q, "bf16", 1, c)),
    "gate, counts too small": (lambda: (*(finite((5, 64), torch.bfloat16, s) for s in (1, 2, 3, 4)), torch.zeros(3, device="cuda", dtype=torch.int32)),
                               lambda y, v, r, q, c: B.addrms_gate_probe_noalloc(y, v, r, q, "bf16", 1, c)),
    "gate, tolerance beyond 32 bits": (lambda: (*(finite((5, 64), torch.bfloat16, s) for s in (1, 2, 3, 4)), torch.zeros(4, device="cuda", dtype=torch.int32)),
                                       lambda y, v, r, q, c: B.addrms_gate_probe_noalloc(y, v, r, q, "bf16", (1 << 32) + 2, c)),
}


@pytest.mark.gpu
@pytest.mark.parametrize("what", CALLS)
def test_both_ways_do_the_same(monkeypatch, what):
    B.addrms_table_clear()
    B._torch()
    make, call = CALLS[what]
    fast, slow = (outcome(monkeypatch, native, make, call) for native in (True, False))
    assert type(fast) is type(slow), (fast, slow)
    if isinstance(fast, tuple):
        assert fast == slow
    else:
        assert all(torch.equal(a, b) for a, b in zip(fast, slow))


@pytest.mark.gpu
def test_the_current_stream_is_the_one_of_the_moment():
    """A call inside a capture is recorded, not run: on any other stream it would run at once."""
    x, r, w = norm()
    B._torch()
    before = bits(x).clone()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        assert B._native.addrms_run(x, r, w, 1e-6, 9, 1000, "bf16", None) == 0
    torch.cuda.synchronize()
    assert torch.equal(bits(x), before)
    graph.replay()
    torch.cuda.synchronize()
    assert not torch.equal(bits(x), before)


@pytest.mark.gpu
def test_a_call_leaves_the_interpreters_lock():
    """The entry point replaced by one that needs the lock (a Python callback): it is called without it, so the callback
    can take it, and its status comes back."""
    B._torch()
    x, r, w = norm()
    seen = []
    fn = ctypes.CFUNCTYPE(ctypes.c_int, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_float, ctypes.c_int64, ctypes.c_int64,
                          ctypes.c_int, ctypes.c_void_p, ctypes.c_void_p)(lambda *a: seen.append(a) or -5)
    lib = B.load()
    real = [ctypes.cast(getattr(lib, f), ctypes.c_void_p).value for f in
            ("addrms_run", "silumul_run", "mergestates_run", "addrms_gate_probe_noalloc")]
    try:
        B._native.bind(B.DTYPE_IDS, B.Cfg, ctypes.cast(fn, ctypes.c_void_p).value, *real[1:])
        assert B._native.addrms_run(x, r, w, 0.25, 9, 1000, "bf16", None) == -5
    finally:
        B._native.bind(B.DTYPE_IDS, B.Cfg, *real)
    assert seen[0][:7] == (x.data_ptr(), r.data_ptr(), w.data_ptr(), 0.25, 9, 1000, 0)
