"""Tiled int8 kernel with 64-row tiles and its slabs (the last wavefront of a strip keeps its own sums), at the edges:
one row in the last tile, strips that leave wavefronts idle, a short last slab, zero-points inside and beyond the codes.

The integer sum inside a part (a chunk of 128 k, or a scale group of 64) is exact; the parts, whatever group they belong to, and
the slabs are added in fp32, one rounding to the output type:
|C - ref| <= u |ref| + 2^-23 (parts + 2) sum_parts s |sum_k a (q - z)|, u = 2^-11 (fp16) or 2^-8 (bf16)."""
import numpy as np
import pytest
import torch

from gpu_util import bits_of

pytestmark = pytest.mark.gpu
K, N = 1408, 320                 # eleven chunks, five strips


@pytest.fixture(autouse=True)
def _reset_knobs():
    yield
    from paper_2504_12984_amd import binding as B
    for k in range(4):
        B.qg_set_knob(k, 0)


@pytest.mark.parametrize("splitk", [1, 2, 3, 5, 8])
@pytest.mark.parametrize("bm,M", [(64, 1), (64, 65), (64, 200), (128, 129)])
@pytest.mark.parametrize("kind,bits,zeros", [("u", 4, "in"), ("i", 8, None), ("u", 7, "beyond"), ("u", 8, "in")])
def test_row_tiles_and_slabs(kind, bits, zeros, bm, M, splitk):
    from paper_2504_12984_amd import binding as B
    gen = torch.Generator(device="cuda").manual_seed(1000 * splitk + M + bits)
    t = B.WType(B.QG_UINT if kind == "u" else B.QG_INT, bits)
    group = (64, 128, K)[(M + splitk) % 3]
    rows = K // group
    out = torch.bfloat16 if splitk % 2 else torch.float16
    codes = torch.randint(0, 1 << bits, (K, N), dtype=torch.uint8, device="cuda", generator=gen)
    packed = B.repack(B.qg_pack_codes(codes, bits), t, K, N, layout=B.QG_LAYOUT_TILE128x64_I8)
    scales = (0.01 + 0.02 * torch.rand(rows, N, device="cuda", generator=gen)).to(out)
    Z = None if zeros is None else torch.randint(0, 256 if zeros == "beyond" else 1 << bits, (rows, N), dtype=torch.uint8, device="cuda", generator=gen)
    A = torch.randint(-128, 128, (M, K), dtype=torch.int8, device="cuda", generator=gen)
    a_scale = 0.01 + 0.01 * torch.rand(M, device="cuda", generator=gen)
    for k, v in enumerate((2, splitk, bm)):
        B.qg_set_knob(k, v)
    C = B.qgemm_a8(A, a_scale, packed, scales, Z, t, group, N, out_dtype=out)
    assert np.array_equal(bits_of(C), bits_of(B.qgemm_a8(A, a_scale, packed, scales, Z, t, group, N, out_dtype=out)))      # counters left clean
    q = codes.cpu().to(torch.int64)
    q = q - ((q >> (bits - 1)) << bits) if kind == "i" else q
    a, s, ref, size = A.cpu().to(torch.int64), scales.cpu().double(), 0.0, 0.0
    part = min(group, 128)
    for k in range(0, K, part):
        g = k // group
        one = torch.mm(a[:, k:k + part], q[k:k + part] - (0 if Z is None else Z[g].cpu().to(torch.int64))).double() * s[g]
        ref, size = ref + one, size + one.abs()
    sa = a_scale.cpu().double()[:, None]
    bound = (2.0 ** -8 if out is torch.bfloat16 else 2.0 ** -11) * (ref * sa).abs() + 2.0 ** -23 * (K // part + 2) * size * sa + 2.0 ** -24
    assert bool(((C.cpu().double() - ref * sa).abs() <= bound).all())
