"""Streaming int8 kernel: two, three and four 16-row tiles at the rows where the choice changes."""
import pytest
import torch

pytestmark = pytest.mark.gpu
K, N = 1408, 320


@pytest.fixture(autouse=True)
def _reset_knobs():
    yield
    from paper_2504_12984_amd import binding as B
    for k in range(4):
        B.qg_set_knob(k, 0)


@pytest.mark.parametrize("M", [32, 33, 40, 48, 49])
@pytest.mark.parametrize("kind,bits,group,kk", [("u", 4, 128, 2176), ("i", 8, 64, K), ("u", 3, 0, K), ("u", 8, 128, 2176)])
def test_rows(kind, bits, group, kk, M):
    """The sum inside a part (a chunk, or a scale group of 64) is an exact integer, the
    parts are added in fp32, one rounding: |C - ref| <= 2^-11 |ref| + 2^-23 (parts + 2) sum_parts s |sum_k a (q - z)|."""
    from paper_2504_12984_amd import binding as B
    gen = torch.Generator(device="cuda").manual_seed(100 * M + bits)
    t = B.WType(B.QG_UINT if kind == "u" else B.QG_INT, bits)
    rows = kk // group if group else 1
    codes = torch.randint(0, 1 << bits, (kk, N), dtype=torch.uint8, device="cuda", generator=gen)
    packed = B.repack(B.qg_pack_codes(codes, bits), t, kk, N, layout=B.QG_LAYOUT_TILE128x64_I8)
    scales = (0.01 + 0.02 * torch.rand(rows, N, device="cuda", generator=gen)).half()
    Z = torch.randint(0, 1 << bits, (rows, N), dtype=torch.uint8, device="cuda", generator=gen) if kind == "u" else None
    A = torch.randint(-128, 128, (M, kk), dtype=torch.int8, device="cuda", generator=gen)
    a_scale = 0.01 + 0.01 * torch.rand(M, device="cuda", generator=gen)
    q = codes.cpu().to(torch.int64)
    q = q - ((q >> (bits - 1)) << bits) if kind == "i" else q
    a, s, ref, size, part = A.cpu().to(torch.int64), scales.cpu().double(), 0.0, 0.0, min(group or kk, 128)
    for k in range(0, kk, part):
        g = k // group if group else 0
        one = torch.mm(a[:, k:k + part], q[k:k + part] - (0 if Z is None else Z[g].cpu().to(torch.int64))).double() * s[g]
        ref, size = ref + one, size + one.abs()
    sa = a_scale.cpu().double()[:, None]
    bound = 2.0 ** -11 * (ref * sa).abs() + 2.0 ** -23 * (kk // part + 2) * size * sa + 2.0 ** -24
    B.qg_set_knob(0, 3)
    for splitk in (1, 3):
        B.qg_set_knob(1, splitk)
        C = B.qgemm_a8(A, a_scale, packed, scales, Z, t, group, N)
        assert bool(((C.cpu().double() - ref * sa).abs() <= bound).all()), splitk
