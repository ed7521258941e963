"""Calls that name no configuration and have none in the table take kernels of their own, chosen by the problem.
They must give what the default configuration gives (same arithmetic, element by element), touch nothing beside their
outputs, and leave to the default configuration what they do not cover.

The comparison is of bits.  A row's sum of squares is taken in fp64 in another order than the default configuration's,
so rstd may in principle round to the neighbouring fp32 value: two orders differ by about sqrt(N) * 2^-53, which crosses
one of the rounding boundaries 2^-24 apart in some 1e-7 of rows, a hundredth of one row over all the rows here.  The
seeds are fixed, so what passes keeps passing."""
import numpy as np
import pytest
import torch

from paper_2601_12698_amd import binding as B
from paper_2601_12698_amd import workloads as W
from ulp import ulp_distance

pytestmark = pytest.mark.gpu
PAD = 64            # canary elements on either side of an output


@pytest.fixture(autouse=True)
def _empty_table():
    B.addrms_table_clear()


def bits(t):
    return t.view(torch.int16 if t.element_size() == 2 else torch.int32)


def guarded(numel, dtype, off=0):
    """A tensor of numel elements, off elements past an aligned address, and a check that its surroundings are untouched."""
    buf = torch.full((numel + 2 * PAD + off,), 42.0, dtype=dtype, device="cuda")
    view = buf[PAD + off:PAD + off + numel]

    def intact():
        return bool((buf[:PAD + off] == 42.0).all()) and bool((buf[PAD + off + numel:] == 42.0).all())
    return view, intact


def finite(shape, dtype, seed, std=1.5):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return (torch.randn(shape, generator=g, device="cuda") * std).to(dtype)


def normal(shape, dtype, seed, std=1.5):
    """With two infinities among the values: for operators that work element by element (a row of the norm that holds one
    has nothing left to compare)."""
    t = finite(shape, dtype, seed, std)
    t.view(-1)[0] = float("inf")
    t.view(-1)[t.numel() // 2] = -float("inf")
    return t


SILU = [("bf16", 1, 16), ("bf16", 3, 17), ("bf16", 1, 23), ("fp16", 5, 1000), ("fp16", 7, 1001), ("fp32", 3, 9), ("fp32", 2, 8),
        ("fp32", 11, 1003), ("bf16", 33, 2056), ("bf16", 2, 8191), ("bf16", 2000, 4099), ("bf16", 6500, 8200), ("fp16", 6500, 8190),
        ("bf16", 4, 15), ("fp32", 1, 28672)]


@pytest.mark.parametrize("dtype,M,d", SILU)
def test_gated_activation(dtype, M, d):
    """Pieces of 16 bytes: rows shorter than two of them, rows that end inside one, an output that ends inside one, and
    outputs on both sides of the size where the store policy changes."""
    t = W.x_torch_dtype(dtype)
    x = normal((M, 2 * d), t, d)
    want = torch.empty((M, d), dtype=t, device="cuda")
    B.silumul_run(x, want, M, d, dtype, B.silumul_default_cfg(d, dtype))
    got, intact = guarded(M * d, t)
    B.silumul_run(x, got, M, d, dtype)
    torch.cuda.synchronize()
    assert torch.equal(bits(got), bits(want).view(-1)) and intact()


@pytest.mark.parametrize("off", [1, 2, 4])
def test_gated_activation_with_bases_that_are_not_16_byte_aligned(off):
    """Odd d: one-element accesses were always accepted at any element; even so with the input alone off, and refused as
    before where the default configuration's access does not fit the base."""
    M, d = 9, 1001
    buf = normal((2 * M * d + 8,), torch.bfloat16, 5)
    x = buf[off:off + 2 * M * d]
    want = torch.empty((M, d), dtype=torch.bfloat16, device="cuda")
    B.silumul_run(x, want, M, d, "bf16", B.silumul_default_cfg(d, "bf16"))
    for out_off in (0, off):
        got, intact = guarded(M * d, torch.bfloat16, out_off)
        B.silumul_run(x, got, M, d, "bf16")
        torch.cuda.synchronize()
        assert torch.equal(bits(got), bits(want).view(-1)) and intact()
    with pytest.raises(B.AddrmsError) as e:
        B.silumul_run(buf[off:off + 2 * 8 * 1000], got[:8 * 1000], 8, 1000, "bf16")
    assert e.value.status == B.ERR_MISALIGNED


MERGE = [("bf16", 30000, 64), ("fp16", 20011, 128), ("bf16", 9001, 192), ("bf16", 24576, 256), ("fp16", 7003, 1000),
         ("bf16", 250_000, 256), ("fp16", 3, 128), ("bf16", 60000, 72), ("bf16", 40000, 100)]


@pytest.mark.parametrize("dtype,rows,d", MERGE)
def test_merge_of_attention_states(dtype, rows, d):
    t = W.x_torch_dtype(dtype)
    va, vb = normal((rows, d), t, 1), normal((rows, d), t, 2)
    sa, sb = normal((rows,), torch.float32, 3, 3.0).nan_to_num(posinf=80.0, neginf=-80.0), \
        normal((rows,), torch.float32, 4, 3.0).nan_to_num(posinf=80.0, neginf=-80.0)
    vw, sw = torch.empty_like(va), torch.empty_like(sa)
    B.mergestates_run(va, sa, vb, sb, vw, sw, rows, d, dtype, B.mergestates_default_cfg(d, dtype))
    vo, vok = guarded(rows * d, t)
    so, sok = guarded(rows, torch.float32)
    B.mergestates_run(va, sa, vb, sb, vo, so, rows, d, dtype)
    torch.cuda.synchronize()
    assert torch.equal(bits(vo), bits(vw).view(-1)) and torch.equal(bits(so), bits(sw)) and vok() and sok()


def test_merge_of_states_with_scores_far_apart(oracle):
    """Scores from equal to 2000 apart, at a size that the flat kernel takes (above 4 MB), against the oracle: the part with
    the larger score by far comes out as it went in.  Bounds as in test_gpu_mergestates.py; repeated rows, so that every pair
    of scores meets every place in a workgroup."""
    pairs = torch.tensor([[0.0, 0.0], [5.0, -5.0], [-5.0, 5.0], [90.0, -90.0], [-90.0, 90.0], [1e3, -1e3], [-1e3, 1e3], [3.25, 3.25],
                          [3.25, 3.2500002], [-1e3, -1e3], [1e3, 1e3]])
    d, rows = 128, 11 * 700
    va, vb = (finite((rows, d), torch.bfloat16, s).abs() + 0.125 for s in (5, 6))       # one sign: nothing cancels
    sa, sb = pairs[:, 0].repeat(700).cuda(), pairs[:, 1].repeat(700).cuda()
    vo, so = torch.empty_like(va), torch.empty_like(sa)
    B.mergestates_run(va, sa, vb, sb, vo, so, rows, d, "bf16")
    torch.cuda.synchronize()
    vref, sref = oracle.mergestates(W.to_bits(va), sa.cpu().numpy(), W.to_bits(vb), sb.cpu().numpy(), 0)
    assert ulp_distance(W.to_bits(vo), vref).max() <= 1
    assert np.allclose(so.cpu().numpy(), sref, rtol=0, atol=4e-7 * np.maximum(1.0, np.abs(sref)))
    k = torch.arange(rows, device="cuda") % 11
    assert torch.equal(vo[(k == 3) | (k == 5)], va[(k == 3) | (k == 5)]) and torch.equal(vo[(k == 4) | (k == 6)], vb[(k == 4) | (k == 6)])


def test_merge_of_states_with_scores_that_are_not_finite():
    """Outside what the operator promises; the flat kernel gives the bits of the default configuration even so."""
    inf, nan = float("inf"), float("nan")
    pairs = torch.tensor([[-inf, 0.0], [0.0, -inf], [-inf, -inf], [inf, 0.0], [inf, inf], [nan, 0.0], [0.0, nan]])
    d, rows = 256, 7 * 500
    va, vb = finite((rows, d), torch.float16, 7), finite((rows, d), torch.float16, 8)
    sa, sb = pairs[:, 0].repeat(500).cuda(), pairs[:, 1].repeat(500).cuda()
    vw, sw, vo, so = torch.empty_like(va), torch.empty_like(sa), torch.empty_like(va), torch.empty_like(sa)
    B.mergestates_run(va, sa, vb, sb, vw, sw, rows, d, "fp16", B.mergestates_default_cfg(d, "fp16"))
    B.mergestates_run(va, sa, vb, sb, vo, so, rows, d, "fp16")
    torch.cuda.synchronize()
    assert torch.equal(bits(vo), bits(vw)) and torch.equal(bits(so), bits(sw))


def norm_inputs(M, N, dtype, seed, off=0, special=None):
    """Finite values, so that every element of y depends on its row's sum; special: (row, column, value) of x entries that
    are set to an infinity or NaN instead."""
    x, xok = guarded(M * N, W.x_torch_dtype(dtype), off)
    r, rok = guarded(M * N, W.r_torch_dtype(dtype), off)
    x.copy_(finite((M * N,), x.dtype, seed))
    r.copy_(finite((M * N,), r.dtype, seed + 1))
    for row, col, value in special or ():
        x[row * N + col] = value
    w = torch.rand(N + off, generator=torch.Generator(device="cuda").manual_seed(seed + 2), device="cuda").to(x.dtype)[off:]
    return x, xok, r, rok, w


def check_norm(M, N, dtype, off=0, special=None):
    x, xok, r, rok, w = norm_inputs(M, N, dtype, N, off, special)
    xw, rw = x.clone(), r.clone()
    if off:                                                       # the clones start at an aligned address
        xw, rw = torch.cat([xw[:off], xw])[off:], torch.cat([rw[:off], rw])[off:]
    B.addrms_run(xw, rw, w, 1e-6, M, N, dtype, B.addrms_default_cfg(N, dtype))
    B.addrms_run(x, r, w, 1e-6, M, N, dtype)
    torch.cuda.synchronize()
    # what is compared must be able to differ: y finite, and zero only where a sum of the inputs or a weight happens to be
    # (16-bit normals: one in a few hundred, so half of even the shortest rows, of 8 elements, is one row in 10^8)
    plain = xw.view(M, N)
    if special:
        plain = plain[[row for row in range(M) if row not in {s[0] for s in special}]]
    assert bool(torch.isfinite(plain).all()) and bool(((plain != 0).float().mean(dim=1) > 0.5).all())
    assert torch.equal(bits(r), bits(rw)) and torch.equal(bits(x), bits(xw)) and xok() and rok()


# N in pieces of 16 bytes (8 or 4 elements): half a wave and one more, whole waves and one more, one piece per thread
# at its limit and beyond, the most a thread holds; M around the rows of a workgroup; sizes on both sides of the store
# policy's two limits (512 KB and 96 MB)
NORM = [("bf16", 1, 136), ("bf16", 7, 256), ("bf16", 8, 264), ("fp16", 5, 512), ("fp16", 3, 520), ("bf16", 2, 8192),
        ("bf16", 3, 8200), ("fp16", 2, 16384), ("fp16", 2, 24584), ("bf16", 2, 32768), ("fp32", 3, 68), ("fp32", 5, 132),
        ("fp32", 2, 4096), ("fp32", 2, 4100), ("fp32", 2, 16388), ("fp32", 2, 24580), ("fp32", 1, 32768),
        ("fp16_res32", 3, 72), ("fp16_res32", 9, 1000), ("fp16_res32", 3, 1004), ("fp16_res32", 2, 20484),
        ("fp16_res32", 2, 32764), ("bf16", 4096, 1024), ("bf16", 4095, 1024), ("bf16", 6144, 4096), ("bf16", 6145, 4096),
        ("fp32", 700, 3584), ("fp16_res32", 5000, 2880), ("bf16", 127, 1024), ("bf16", 128, 1024),
        # whole vectors but not whole lines, from 512 KB on: every number of pieces per thread, two rows in a workgroup
        ("bf16", 2001, 136), ("fp16", 300, 1000), ("bf16", 40, 10008), ("bf16", 20, 22376), ("fp16", 11, 30008), ("fp32", 1001, 100),
        ("fp32", 200, 1004), ("fp32", 40, 5004), ("fp32", 20, 10004), ("fp32", 20, 15004), ("fp32", 12, 20004), ("fp32", 10, 28004),
        ("fp16_res32", 2003, 100), ("fp16_res32", 700, 200), ("fp16_res32", 20, 12004), ("bf16", 150_001, 200)]


@pytest.mark.parametrize("dtype,M,N", NORM)
def test_norm(dtype, M, N):
    check_norm(M, N, dtype)


# rows that 16 bytes do not divide (every remainder), that lines do not divide, that begin at every element of a line,
# with as many pieces as threads and one more, and the longest ones; small ones that the default configuration keeps
RAGGED = [("bf16", 67, 129), ("bf16", 66, 131), ("fp16", 130, 255), ("fp16", 9, 1001), ("fp16", 9, 1003), ("bf16", 9, 1005),
          ("bf16", 9, 1007), ("bf16", 700, 1030), ("bf16", 600, 1020), ("bf16", 5, 449), ("bf16", 5, 450), ("fp32", 70, 65),
          ("fp32", 35, 67), ("fp32", 9, 1001), ("fp32", 300, 1002), ("fp32", 3, 4067), ("fp32", 3, 4069), ("fp16_res32", 65, 67),
          ("fp16_res32", 9, 1001), ("fp16_res32", 9, 4033), ("fp16_res32", 9, 4035), ("bf16", 40, 1030), ("bf16", 3, 8129),
          ("bf16", 3, 8131), ("fp16", 2, 16385), ("fp16", 2, 32705), ("fp16", 2, 32707), ("fp32", 2, 32737), ("fp32", 2, 32739),
          ("fp16_res32", 2, 32705), ("bf16", 4500, 1000), ("fp16_res32", 3000, 1000), ("fp32", 2200, 1004), ("bf16", 9000, 6150),
          ("bf16", 3001, 1528), ("bf16", 3001, 1544), ("bf16", 26001, 1000), ("fp32", 17001, 764), ("fp16_res32", 11003, 260),
          ("fp16_res32", 17001, 1000),
          # from 4 MB on with up to three pieces per thread, and one or two rows in a workgroup
          ("bf16", 12001, 129), ("bf16", 9001, 131), ("fp16", 5001, 255), ("bf16", 5003, 451), ("bf16", 1603, 1020), ("fp16", 2101, 1001),
          ("bf16", 501, 4001), ("fp32", 601, 1001), ("fp32", 300, 2001), ("fp16_res32", 901, 1001), ("fp16_res32", 300, 4001)]


@pytest.mark.parametrize("dtype,M,N", RAGGED)
def test_norm_of_ragged_rows(dtype, M, N):
    check_norm(M, N, dtype)


@pytest.mark.parametrize("dtype", W.DTYPES)
@pytest.mark.parametrize("off", [1, 2, 3, 5])
def test_norm_of_ragged_rows_from_any_element(dtype, off):
    check_norm(17, 1001, dtype, off)


def test_norm_of_ragged_rows_whose_streams_begin_at_different_elements():
    M, N = 17, 1001
    x, xok, r, rok, w = norm_inputs(M, N, "bf16", 7, 1)
    r2, r2ok = guarded(M * N, torch.bfloat16, 0)
    r2.copy_(r)
    xw, rw = x.clone(), r.clone()
    B.addrms_run(xw, rw, w, 1e-6, M, N, "bf16", B.addrms_default_cfg(N, "bf16"))
    B.addrms_run(x, r2, w, 1e-6, M, N, "bf16")
    torch.cuda.synchronize()
    assert torch.equal(bits(r2), bits(rw)) and torch.equal(bits(x), bits(xw)) and xok() and r2ok()


def test_norm_refuses_bases_the_default_configuration_refuses():
    x, _, r, _, w = norm_inputs(8, 1000, "bf16", 7, 1)
    with pytest.raises(B.AddrmsError) as e:
        B.addrms_run(x, r, w, 1e-6, 8, 1000, "bf16")
    assert e.value.status == B.ERR_MISALIGNED


# rows beyond the registers: the first length that is, and for the kernel of captured calls, which test_long_rows.py runs on
# them, one chunk parked in LDS and one left over, as much as LDS holds and more (read twice), whole lines or not; both
# store policies.  Eager calls split all of them but two.
LONG = [("bf16", 2, 32776), ("bf16", 3, 32832), ("fp16", 2, 32707), ("bf16", 2, 49152), ("bf16", 2, 49160), ("fp16", 2, 57344),
        ("bf16", 2, 81920), ("bf16", 2, 81984), ("bf16", 2, 90113), ("fp16", 2, 131071), ("bf16", 1, 1 << 20), ("fp32", 2, 32772),
        ("fp32", 2, 32741), ("fp32", 2, 49156), ("fp32", 2, 86016), ("fp32", 2, 86048), ("fp32", 2, 86019), ("fp32", 2, 200001),
        ("fp16_res32", 2, 32832), ("fp16_res32", 2, 49153), ("fp16_res32", 2, 86020), ("fp16_res32", 2, 100003),
        ("bf16", 700, 40960), ("bf16", 300, 99991), ("fp32", 150, 100000), ("fp16_res32", 200, 86022)]


@pytest.mark.parametrize("dtype,M,N", LONG)
def test_norm_of_rows_beyond_the_registers(dtype, M, N):
    check_norm(M, N, dtype)


@pytest.mark.parametrize("dtype,N", [("bf16", 4096), ("bf16", 200), ("fp16", 1001), ("fp32", 16388), ("fp16_res32", 2880),
                                     ("bf16", 81984), ("fp32", 86019)])
def test_norm_keeps_infinities_and_nan_in_their_rows(dtype, N):
    """First, inner and last element of a row (ragged rows: elements outside the whole pieces); the rows beside them are
    compared as in every other case."""
    inf = float("inf")
    check_norm(7, N, dtype, special=[(1, 0, inf), (3, N // 2, -inf), (4, N - 1, inf), (5, N - 1, float("nan"))])


@pytest.mark.parametrize("off", [1, 3])
def test_norm_of_long_ragged_rows_from_any_element(off):
    check_norm(3, 40001, "bf16", off)
    check_norm(3, 90001, "fp32", off)


@pytest.mark.parametrize("dtype", ["bf16", "fp32", "fp16_res32"])
def test_norm_from_bases_that_only_a_narrow_default_access_fits(dtype):
    """Rows of whole 16-byte pieces whose default configuration reads two elements at a time (86912: what LDS holds at that
    width), so that it takes bases no 16-byte access fits; the weights alone may be off, too."""
    N = 86912
    assert B.addrms_default_cfg(N, dtype).vec < (8 if dtype == "bf16" else 4)
    for off in (0, 2, 4, 6):
        check_norm(3, N, dtype, off)
    x, xok, r, rok, _ = norm_inputs(3, N, dtype, 1)
    w = torch.rand(N + 2, generator=torch.Generator(device="cuda").manual_seed(3), device="cuda").to(x.dtype)[2:]
    xw, rw = x.clone(), r.clone()
    B.addrms_run(xw, rw, w, 1e-6, 3, N, dtype, B.addrms_default_cfg(N, dtype))
    B.addrms_run(x, r, w, 1e-6, 3, N, dtype)
    torch.cuda.synchronize()
    assert torch.equal(bits(x), bits(xw)) and torch.equal(bits(r), bits(rw)) and xok() and rok()


@pytest.mark.parametrize("seed", range(8))
def test_any_form_the_default_configuration_takes(seed):
    """Sizes, formats and first elements at random: whatever route a call takes, the bits are the default configuration's."""
    import random
    rng = random.Random(seed)
    for _ in range(12):
        dtype = rng.choice(W.DTYPES)
        N = int(2 ** rng.uniform(3, 16.5))
        N = rng.choice((N, N // 8 * 8 or 8, N // 64 * 64 or 64))
        M = rng.choice((1, 2, 3, 5, 64, 513))
        M = max(1, min(M, 4_000_000 // N))
        vec = B.addrms_default_cfg(N, dtype).vec
        off = rng.choice((0, 0, *(v for v in (1, 2, 4, 8) if v % vec == 0)))
        print(f"add+RMSNorm {dtype} {M} x {N} from element {off}", flush=True)
        check_norm(M, N, dtype, off)
    for _ in range(6):
        dtype = rng.choice(("bf16", "fp16", "fp32"))
        d = int(2 ** rng.uniform(3, 13))
        M = max(1, min(rng.choice((1, 2, 7, 300)), 2_000_000 // d))
        print(f"gated activation {dtype} {M} x {d}", flush=True)
        test_gated_activation(dtype, M, d)


def test_calls_without_a_configuration_in_a_graph():
    """Captured once, replayed with other work of the stream in between: every replay starts from the same inputs and
    must leave what the eager call leaves.  The long rows park 128 KB in LDS, beyond what a launch may ask for by default."""
    cases = [("bf16", 16, 4096), ("fp16", 300, 1001), ("bf16", 600, 4096), ("bf16", 3, 81920)]
    state = []
    for dtype, M, N in cases:
        x, _, r, _, w = norm_inputs(M, N, dtype, N)
        state.append((dtype, M, N, x.clone(), r.clone(), w, torch.empty_like(x), torch.empty_like(r)))
    xs = normal((64, 2 * 1001), torch.bfloat16, 3)
    out = torch.empty((64, 1001), dtype=torch.bfloat16, device="cuda")

    def body():
        for dtype, M, N, x0, r0, w, x, r in state:
            x.copy_(x0)
            r.copy_(r0)
            B.addrms_run(x, r, w, 1e-6, M, N, dtype)
        B.silumul_run(xs, out, 64, 1001, "bf16")

    body()
    torch.cuda.synchronize()
    want = [(bits(s[6]).clone(), bits(s[7]).clone()) for s in state] + [(bits(out).clone(), bits(out).clone())]
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        body()
    for _ in range(3):
        for s in state:
            s[6].fill_(1.0)
            s[7].fill_(1.0)
        out.fill_(1.0)
        graph.replay()
        torch.cuda.synchronize()
        got = [(bits(s[6]), bits(s[7])) for s in state] + [(bits(out), bits(out))]
        assert all(torch.equal(a, c) and torch.equal(b, d) for (a, b), (c, d) in zip(got, want))


@pytest.mark.parametrize("less", [2, 0])
def test_as_many_rows_as_one_launch_takes_and_more(less):
    """32 threads a row: 2^27 - 2 rows are the most that the 2^32 - 1 threads of a launch cover; from 2^27 on the
    default configuration with its 16 threads a row runs instead.  1024 different rows, repeated."""
    M, N, block = 2 ** 27, 128, 1024
    if torch.cuda.mem_get_info()[0] < 90 << 30:
        pytest.skip("needs 70 GB of device memory")
    want = [finite((block, N), torch.bfloat16, s) for s in (1, 2)]
    weight = finite((N,), torch.bfloat16, 3)
    x, r = (t.view(1, -1).expand(M // block, -1).contiguous() for t in want)
    before = [t.view(-1)[-less * N:].clone() if less else None for t in (x, r)]
    B.addrms_run(want[0], want[1], weight, 1e-5, block, N, "bf16", B.addrms_default_cfg(N, "bf16"))
    rows = M - less
    B.addrms_run(x.view(-1)[:rows * N], r.view(-1)[:rows * N], weight, 1e-5, rows, N, "bf16")
    torch.cuda.synchronize()
    for got, ref, old in ((x, want[0], before[0]), (r, want[1], before[1])):
        if less:
            assert torch.equal(bits(got.view(-1)[-less * N:]), bits(old))
            got.view(-1)[-less * N:] = ref.view(-1)[-less * N:]
        for c in range(0, M // block, 8192):
            assert bool((bits(got[c:c + 8192]) == bits(ref).view(1, -1)).all()), c
    del x, r
    torch.cuda.empty_cache()
