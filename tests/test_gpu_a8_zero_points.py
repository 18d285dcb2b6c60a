"""Zero-points in the tiled int8 kernel: code and zero-point cancel inside a scale group, so the sum over the group
has to be an exact integer there as it is in the streaming kernel.  Long K, activations with a mean, codes
at or near zero-points far from the middle, zero-points beyond the codes (in all columns, or in a few).

Bound: with the integers t of a chunk (min(group, 128) rows) exact, one fp32 rounding per chunk and one for the
row scale, |C - ref| <= u |ref| + (chunks + 1) 2^-24 a_scale sum |s t|, u = 2^-11 (fp16) or 2^-8 (bf16) for the
rounding to the output type (and 2^-24 for fp16 results below its normal range).  Where every code is
its zero-point the result is zero."""
import os
import subprocess
import sys

import numpy as np
import pytest
import torch

from oracle import qgemm_oracle as O
from paper_2504_12984_amd import workloads as WL
from gpu_util import to_f64
from test_gpu_a8 import A8Case, _case, _reset_knobs, I, U  # noqa: F401

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
M, K, N = 130, 8192, 256


def _inputs(case, codes, zeros):
    """codes, zeros: functions of (generator, zeros or codes drawn so far)."""
    c, rng = case, np.random.Generator(np.random.PCG64(case.seed))
    inp = WL.make_inputs(c)
    inp["A"] = torch.from_numpy(np.clip(np.round(rng.standard_normal((c.M, c.K)) * 40 + 30), -128, 127).astype(np.int8))
    z = zeros(rng, (c.K // c.group, c.N))
    inp["zeros"] = z
    full = np.zeros((c.K, c.N), np.int64) if z is None else np.repeat(z.astype(np.int64), c.group, 0)
    q = np.clip(codes(rng, full), 0, (1 << c.bits) - 1) if c.kind == U else codes(rng, full) & ((1 << c.bits) - 1)
    inp["codes"] = q.astype(np.uint8)
    return inp


def _check(P):
    c = P.case
    got, ref = to_f64(P.gpu()), P.ref()
    w = O.int_weights(P.inp["codes"], c.kind, c.bits, P.inp["zeros"], c.group).astype(np.float64)
    A, step = P.inp["A"].numpy().astype(np.float64), min(c.group, 128)
    size = np.zeros(ref.shape)
    for k in range(0, c.K, step):
        size += np.abs(A[:, k:k + step] @ w[k:k + step]) * np.abs(P.S64[k // c.group])[None, :]
    size *= P.inp["a_scale"].numpy().astype(np.float64)[:, None]
    u = 2.0 ** -11 if c.act == "f16" else 2.0 ** -8
    bound = u * np.abs(ref) + (c.K // step + 1) * 2.0 ** -24 * size + 2.0 ** -24
    bad = np.argwhere(~(np.abs(got - ref) <= bound))
    i = tuple(bad[0]) if len(bad) else None
    assert i is None, f"{c.name}: {len(bad)} of {ref.size} outside, first at {i}: {got[i]} for {ref[i]}, bound {bound[i]}"


def _const(v):
    return lambda rng, shape: np.full(shape, v, np.uint8)


def _random(lo, hi):
    return lambda rng, shape: rng.integers(lo, hi + 1, size=shape).astype(np.uint8)


def _few(lo, hi, beyond):      # four zero-points beyond the codes, in one wavefront's columns of groups in the middle
    def draw(rng, shape):
        z = rng.integers(lo, hi + 1, size=shape).astype(np.uint8)
        z[shape[0] // 2:, 70:74] = beyond
        return z
    return draw


def _near(d):
    return lambda rng, z: z + rng.integers(-d, d + 1, size=z.shape)


def _any(rng, z):
    return rng.integers(0, 256, size=z.shape)


CASES = {
    "u8_no_zeros_all_zero": (U, 8, lambda rng, shape: None, _near(0)),
    "u8_at_250": (U, 8, _const(250), _near(0)),
    "u8_near": (U, 8, _random(100, 200), _near(2)),
    "u8_at_128": (U, 8, _const(128), _near(1)),
    "u4_no_zeros_all_zero": (U, 4, lambda rng, shape: None, _near(0)),
    "u4_at_0": (U, 4, _const(0), _near(0)),
    "u4_beyond": (U, 4, _const(250), _any),
    "u4_near": (U, 4, _random(0, 15), _near(1)),
    "u4_few_beyond": (U, 4, _few(0, 15, 255), _near(1)),
    "u4_one_beyond": (U, 4, _few(0, 15, 16), _near(1)),
    "u1_near": (U, 1, _random(0, 1), _near(0)),
    "u3_near": (U, 3, _random(0, 7), _near(1)),
    "u7_near": (U, 7, _random(0, 127), _near(1)),
    "i4_near": (I, 4, _random(0, 7), _near(1)),
    "i4_beyond": (I, 4, _random(0, 15), _any),
    "i8_zeros": (I, 8, _random(0, 127), _near(1)),
    "i8_beyond": (I, 8, _const(255), lambda rng, z: np.full(z.shape, 128)),
}


@pytest.mark.parametrize("group,act", [(64, "f16"), (128, "bf16"), (K, "f16")])
@pytest.mark.parametrize("name", CASES)
def test_code_and_zero_point_cancel_exactly(name, group, act):
    from paper_2504_12984_amd import binding as B
    B.qg_set_knob(0, 2)                                   # (two tiles: blocks of 64 rows would be chosen)
    kind, bits, zeros, codes = CASES[name]
    case = _case(f"a8z_{name}_{group}", M, K, N, kind, bits, group, act=act, seed=42000 + group + bits)
    _check(A8Case(case, _inputs(case, codes, zeros)))


@pytest.mark.parametrize("splitk", [2, 5])
def test_slabs(splitk):
    from paper_2504_12984_amd import binding as B
    B.qg_set_knob(0, 2); B.qg_set_knob(1, splitk)
    for name in ("u8_near", "u4_few_beyond"):
        kind, bits, zeros, codes = CASES[name]
        case = _case(f"a8z_split_{name}", 129, 2048, 192, kind, bits, 128, seed=42100)
        _check(A8Case(case, _inputs(case, codes, zeros)))


@pytest.mark.parametrize("bits", [2, 8])
@pytest.mark.parametrize("zero", ["random", None])
def test_scales_at_the_ends_of_their_range(bits, zero):
    # as the streaming kernel does it: no factor of the tiled kernel's own may overflow or be lost
    from paper_2504_12984_amd import binding as B
    kind = U if zero else I
    case = _case(f"a8z_scales_{bits}_{kind}", 70, 256, 128, kind, bits, 128, act="bf16", zero=zero, seed=42200 + bits)
    inp = WL.make_inputs(case)
    s = inp["scales"].float()
    for col, v in enumerate((2.0 ** (115 if bits == 2 else 108), 2.0 ** -126, 2.0 ** -132, 0.0, float("inf"), float("nan"))):
        s[:, col] = v
    inp["scales"] = s.to(torch.bfloat16)
    inp["a_scale"] = torch.full((70,), 2.0 ** -4)
    P = A8Case(case, inp)
    B.qg_set_knob(0, 2)
    got = P.gpu().float().cpu()
    B.qg_set_knob(0, 3)
    want = P.gpu().float().cpu()
    assert torch.equal(torch.isnan(got), torch.isnan(want)) and torch.equal(torch.isinf(got), torch.isinf(want))
    fin = torch.isfinite(want)
    assert (want[:, 0][fin[:, 0]] != 0).any() and (want[:, 1] != 0).any()
    # two chunks, each rounded once in fp32, and one step of bf16 (2^-133 below its normal range)
    assert ((got - want).abs()[fin] <= 2.0 ** -7 * want.abs()[fin] + 2.0 ** -133).all()


CAPTURE = """
import torch
from paper_2504_12984_amd import binding as B
M, K, N = 300, 8192, 2048
g = torch.Generator().manual_seed(1)
codes = torch.randint(0, 16, (K, N), dtype=torch.uint8, generator=g).cuda()
t = B.WType(B.QG_UINT, 4)
packed = B.repack(B.qg_pack_codes(codes, 4), t, K, N, layout=B.QG_LAYOUT_TILE128x64_I8)
A = torch.randint(-128, 128, (M, K), dtype=torch.int8, generator=g).cuda()
scales, out = torch.full((K // 128, N), 0.01, dtype=torch.float16, device="cuda"), torch.zeros(M, N, dtype=torch.float16, device="cuda")
call = lambda: B.qgemm_a8(A, None, packed, scales, None, t, 128, N, out=out)
want = (A.cpu().float() @ codes.cpu().float()) * scales[0, 0].item()
torch.cuda.synchronize()
side = torch.cuda.Stream()                            # nothing has run on it: no workspace
graph = torch.cuda.CUDAGraph()
with torch.cuda.graph(graph, stream=side):
    call()
def check():
    torch.cuda.synchronize()
    assert ((out.cpu().float() - want).abs() <= 1e-2 + 5e-3 * want.abs()).all()
for _ in range(3):
    out.zero_()
    graph.replay()
    check()
    out.zero_()
    with torch.cuda.stream(side):
        call()                                        # eager, split: makes the workspace
    check()
print("captured")
"""


def test_capture_of_a_call_that_would_split_k_on_a_stream_without_a_workspace():
    r = subprocess.run([sys.executable, "-c", CAPTURE], capture_output=True, text=True, timeout=100, cwd=ROOT)
    assert r.returncode == 0 and "captured" in r.stdout, r.stderr[-2000:]


def test_more_rows_than_one_launch_takes():
    # K = 2^23: 128 rows of A to a launch (32-bit offsets), the last two are a second one; uint1 against the sum of A's
    # bytes where the code is set, in int64 on the GPU
    from paper_2504_12984_amd import binding as B
    M, K, N = 130, 1 << 23, 64
    gen = torch.Generator(device="cuda")
    gen.manual_seed(43000)
    A = torch.randint(-128, 128, (M, K), dtype=torch.int8, device="cuda", generator=gen)
    codes = torch.randint(0, 2, (K, N), dtype=torch.uint8, device="cuda", generator=gen)
    t = B.WType(B.QG_UINT, 1)
    packed = B.repack(B.qg_pack_codes(codes, 1), t, K, N, layout=B.QG_LAYOUT_TILE128x64_I8)
    scales = torch.full((1, N), 2.0 ** -10, dtype=torch.bfloat16, device="cuda")
    B.qg_set_knob(0, 2)
    got = B.qgemm_a8(A, None, packed, scales, None, t, K, N, out_dtype=torch.bfloat16).double()
    want, size = torch.zeros(M, N, device="cuda", dtype=torch.float64), torch.zeros(M, N, device="cuda", dtype=torch.float64)
    rows = [0, 1, 127, 128, 129]
    for m in rows:
        for n in (0, 17, 63):
            x = torch.where(codes[:, n] != 0, A[m], torch.zeros_like(A[m]))
            want[m, n] = x.sum(dtype=torch.int64)
            size[m, n] = x.view(-1, 128).sum(1, dtype=torch.int64).abs().sum()
    bound = 2.0 ** -10 * (2.0 ** -8 * want.abs() + (K // 128 + 1) * 2.0 ** -24 * size)
    cols = torch.tensor([0, 17, 63], device="cuda")
    rows = torch.tensor(rows, device="cuda")
    pick = lambda x: x[rows][:, cols]      # noqa: E731
    assert (pick((got - want * 2.0 ** -10).abs()) <= pick(bound)).all()
