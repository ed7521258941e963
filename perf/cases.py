"""The work that a serving program has this library do, as cases that can be timed and checked.

Every case is one call of a public entry point of ``paper_2601_12698_amd.binding``: the fused residual-add +
RMSNorm in place (``addrms_run``), the gated activation (``silumul_run``), the merge of two partial attention
states (``mergestates_run``), and the comparison of an output pair with a reference pair that stands in front of
every tuned configuration (``addrms_gate_probe_noalloc``).  Shapes are those of the package's workloads and of the
shape lists its tests hold, or plain sizes between them; ``draw`` spreads over the same ranges.

``plan`` is the configuration a program got from the search earlier and saved; without one the call passes none
and runs what the library picks for the shape.
"""
from __future__ import annotations

import math

import torch

from paper_2601_12698_amd import binding as B
from paper_2601_12698_amd import workloads as W

EPS = 1e-6

# (op, dtype, row length, plan): rows of saved tables, vec, threads per row, rows per workgroup, reduce, unroll,
# flags, waves per SIMD, walk
SAVED = (
    ("addrms", "bf16", 7168, "8,448,1,0,1,34,6,0"),
    ("addrms", "bf16", 8192, "8,1024,1,0,1,2,0,0"),
    ("addrms", "fp16_res32", 5120, "2,512,1,0,2,34,0,0"),
    ("addrms", "fp16_res32", 2880, "4,384,1,0,2,2,0,0"),
    ("silumul", "bf16", 11008, "8,704,1,0,1,2,0,0"),
)


def _case(name, op, M, N, dtype, plan="", outliers=0.0):
    return {"name": name, "op": op, "M": M, "N": N, "dtype": dtype, "plan": plan, "outliers": outliers}


def listed():
    return [
        # a handful of tokens through a norm: the smallest call, bound by the call itself and one launch
        _case("norm_16x4096_bf16", "addrms", 16, 4096, "bf16"),
        # a decode step of 64 sequences
        _case("norm_64x8192_bf16", "addrms", 64, 8192, "bf16"),
        # a prefill chunk
        _case("norm_4096x4096_bf16", "addrms", 4096, 4096, "bf16"),
        # the largest prefill, activations with outliers, run with the configuration a search saved for it
        _case("norm_32768x7168_bf16_saved", "addrms", 32768, 7168, "bf16", "8,448,1,0,1,34,6,0", 0.01),
        # half-precision activations beside an fp32 residual stream, rows that are not whole cache lines
        _case("norm_8192x1000_fp16_res32", "addrms", 8192, 1000, "fp16_res32"),
        # a row length that no vector access divides
        _case("norm_2047x4095_fp16", "addrms", 2047, 4095, "fp16"),
        # full precision, a shape of the published fp32 list
        _case("norm_2048x8192_fp32", "addrms", 2048, 8192, "fp32"),
        # rows longer than the registers of a workgroup hold
        _case("norm_1024x131072_bf16", "addrms", 1024, 131072, "bf16"),
        # the gated activation of a prefill chunk and of a decode step
        _case("gate_act_4096x11008_bf16", "silumul", 4096, 11008, "bf16"),
        _case("gate_act_64x14336_fp16", "silumul", 64, 14336, "fp16"),
        # 768 tokens x 32 heads of 256: merging the two halves of a split-context attention
        _case("merge_24576x256_bf16", "merge", 768 * 32, 256, "bf16"),
        # the check of a prefill-sized output pair against its reference
        _case("check_4096x4096_bf16", "check", 4096, 4096, "bf16"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _width(rng, lo, hi):
    n = _log(rng, lo, hi)
    how = rng.random()
    if how < 0.55:
        return max(64, n // 64 * 64)
    if how < 0.8:
        return max(8, n // 8 * 8)
    return n


def draw(rng):
    op = rng.choices(("addrms", "silumul", "merge", "check"), (5, 2, 2, 1))[0]
    if op in ("addrms", "silumul") and rng.random() < 0.15:
        _, dtype, N, plan = rng.choice([s for s in SAVED if s[0] == op])
        return _draw(op, _log(rng, 64, 20000), N, dtype, plan)
    if op == "addrms":
        dtype = rng.choice(W.DTYPES)
        N = _width(rng, 256, 32768) if rng.random() < 0.85 else _width(rng, 32769, 200000)
        M = _log(rng, 1, 40000)
    elif op == "silumul":
        dtype = rng.choice(("bf16", "fp16", "fp32"))
        N, M = _width(rng, 512, 28672), _log(rng, 1, 16384)
    elif op == "merge":
        dtype = rng.choice(("bf16", "fp16"))
        N, M = rng.choice((64, 80, 96, 128, 192, 256)), _log(rng, 32, 1024) * rng.choice((8, 16, 32, 40, 64))
    else:
        dtype = rng.choice(W.DTYPES)
        N, M = _width(rng, 256, 8192), _log(rng, 16, 8192)
    return _draw(op, M, N, dtype, "")


def _draw(op, M, N, dtype, plan):
    # a row length that only narrow accesses divide runs several times longer for its bytes
    most = 4.0e8 if N % 8 == 0 else 1.0e8
    c = {"op": op, "M": M, "N": N, "dtype": dtype, "plan": plan, "outliers": 0.0}
    per_row = work(dict(c, M=1))["bytes"]
    c["M"] = max(1, min(M, int(most / per_row)))
    return c


def _inputs(case, seed):
    op, M, N, dtype = case["op"], case["M"], case["N"], case["dtype"]
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    xt, rt = W.x_torch_dtype(dtype), W.r_torch_dtype(dtype)

    def normal(shape, to, std=1.0):
        return (torch.randn(shape, generator=g, device="cuda", dtype=torch.float32) * std).to(to)

    if op == "addrms":
        x = normal((M, N), xt)
        if case["outliers"]:
            hit = torch.rand((M, N), generator=g, device="cuda", dtype=torch.float32) < case["outliers"]
            x = torch.where(hit, normal((M, N), xt, 50.0), x)
        r = normal((M, N), rt)
        w = (torch.rand((N,), generator=g, device="cuda") + 0.5).to(xt)
        return {"x": x, "r": r, "w": w}
    if op == "silumul":
        return {"x": normal((M, 2 * N), xt, 1.5)}
    if op == "merge":
        return {"va": normal((M, N), xt), "vb": normal((M, N), xt),
                "sa": normal((M,), torch.float32, 3.0), "sb": normal((M,), torch.float32, 3.0)}
    # an output pair and its reference: equal but for a few units in the last place here and there
    y, r = normal((M, N), xt), normal((M, N), rt)
    yi = y.view(torch.int16 if y.element_size() == 2 else torch.int32)
    ri = r.view(torch.int16 if r.element_size() == 2 else torch.int32)
    few = max(1e-5, 200.0 / (M * N))
    off = (torch.rand((M, N), generator=g, device="cuda") < few).to(yi.dtype)
    far = (torch.rand((M, N), generator=g, device="cuda") < few).to(yi.dtype)
    bad = (torch.rand((M, N), generator=g, device="cuda") < few).to(ri.dtype)
    return {"y": (yi + off + 2 * far).view(xt), "y_ref": y, "r": (ri ^ bad).view(rt), "r_ref": r}


def prepare(case, seed):
    s = _inputs(case, seed)
    op, M, N = case["op"], case["M"], case["N"]
    s["case"] = dict(case)
    s["cfg"] = None
    if case["plan"]:
        s["cfg"] = B.Cfg(*(int(v) for v in case["plan"].split(",")))
    if op == "silumul":
        s["out"] = torch.empty((M, N), device="cuda", dtype=s["x"].dtype)
    elif op == "merge":
        s["vo"], s["so"] = torch.empty_like(s["va"]), torch.empty_like(s["sa"])
    elif op == "check":
        s["counts"] = torch.empty(4, device="cuda", dtype=torch.int32)
    return s


def run(s):
    c = s["case"]
    op, M, N, dtype = c["op"], c["M"], c["N"], c["dtype"]
    if op == "addrms":
        B.addrms_run(s["x"], s["r"], s["w"], EPS, M, N, dtype, s["cfg"])
        return s["x"], s["r"]
    if op == "silumul":
        B.silumul_run(s["x"], s["out"], M, N, dtype, s["cfg"])
        return s["out"]
    if op == "merge":
        B.mergestates_run(s["va"], s["sa"], s["vb"], s["sb"], s["vo"], s["so"], M, N, dtype, s["cfg"])
        return s["vo"], s["so"]
    B.addrms_gate_probe_noalloc(s["y"], s["y_ref"], s["r"], s["r_ref"], dtype, 1, s["counts"])
    return s["counts"]


def exact(case, seed):
    s = _inputs(case, seed)
    op, M, N = case["op"], case["M"], case["N"]
    if op == "addrms":
        # the sum of the two streams is formed in fp32 by definition; everything after it here in 64 bits
        h = s["x"].double().add_(s["r"].double())
        del s["x"], s["r"]
        scale = (torch.linalg.vector_norm(h, dim=1, keepdim=True).square_().div_(N).add_(EPS)).rsqrt_()
        y = h * scale
        y *= s["w"].double()
        return y, h
    if op == "silumul":
        g = s["x"][:, :N].double()
        return g.div_(1.0 + torch.exp(-g)).mul_(s["x"][:, N:].double())
    if op == "merge":
        sa, sb = s["sa"].double(), s["sb"].double()
        so = torch.logaddexp(sa, sb)
        vo = s["va"].double() * torch.exp(sa - so)[:, None] + s["vb"].double() * torch.exp(sb - so)[:, None]
        return vo, so

    def ordered(t):
        i = t.view(torch.int16 if t.element_size() == 2 else torch.int32).long()
        top = 1 << (8 * t.element_size() - 1)
        return torch.where(i < 0, -(i + top), i)

    d = (ordered(s["y"]) - ordered(s["y_ref"])).abs()
    it = torch.int16 if s["r"].element_size() == 2 else torch.int32
    bad = (s["r"].view(it) != s["r_ref"].view(it)).sum()
    return torch.stack([bad, (d > 1).sum(), d.max(), torch.zeros_like(bad)]).to(torch.int32)


def work(case):
    op, M, N, dtype = case["op"], case["M"], case["N"], case["dtype"]
    if op == "addrms":
        return {"bytes": W.algorithmic_bytes(M, N, dtype), "flops": 5 * M * N}
    if op == "silumul":
        return {"bytes": W.silumul_algorithmic_bytes(M, N, dtype), "flops": 5 * M * N}
    if op == "merge":
        return {"bytes": W.merge_algorithmic_bytes(M, N, dtype), "flops": 3 * M * N}
    return {"bytes": 2 * M * N * (W.x_bytes(dtype) + W.r_bytes(dtype)) + 16, "flops": 2 * M * N}


def tolerance(case):
    # Four times the distance between the path and exact(), which is the rounding into the storage format:
    # 1.7e-3 of the norm and half a unit in the last place in bf16, 2.1e-4 in fp16, and in fp32 a few units of
    # the sums, exponentials and reciprocals.
    if case["op"] == "check":
        return "exact"
    if case["dtype"] == "fp32":
        return {"rel": 1e-6, "max": 1e-5}
    if case["dtype"] == "bf16":
        return {"rel": 7e-3, "max": 1.6e-2}
    return {"rel": 8.5e-4, "max": 2e-3}
