"""Tiled kernels: row tiles of 128 and of 64 in one launch.  A last row tile of at most 64 rows, 128-row tiles computed as two
halves, both, more than one round of either (the lower ones among the others, or behind them), 256-row tiles with such a launch
behind, strips that leave wavefronts idle.

An output's sums run over k in the same order whatever its tile, so they equal those of 64-row tiles bit for bit; those
are held against the oracle: |C - ref| <= u |ref| + K 2^-24 sum |a w| (fp32 sums), u = 2^-11 (fp16) or 2^-8 (bf16)."""
import numpy as np
import pytest
import torch

from paper_2504_12984_amd import workloads as WL
from gpu_util import Prepared, bits_of, to_f64

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _reset_knobs():
    yield
    from paper_2504_12984_amd import binding as B
    for k in range(4):
        B.qg_set_knob(k, 0)


# (columns, rows): see the first paragraph; 16384 columns are 64 column tiles, 16448 one more with a single strip
@pytest.mark.parametrize("N,M", [(16384, 257), (16448, 320), (16384, 600), (16448, 700), (16384, 705), (16448, 1100), (16384, 1600)])
def test_mixed_heights(N, M):
    from paper_2504_12984_amd import binding as B
    act = "f16" if M % 2 else "bf16"
    P = Prepared(WL.Case(f"mixed_{N}_{M}", M, 256, N, WL.KIND_UINT, 3 + M % 3, group=(64, 128)[M % 2], act=act, scale_dtype=act,
                         zero="random", zero_hi=7, seed=61000 + M))
    B.qg_set_knob(0, 2)
    got = P.gpu_c()
    B.qg_set_knob(2, 64)
    assert np.array_equal(bits_of(got), bits_of(P.gpu_c()))
    W, _ = P.oracle_w()
    rows = np.unique(np.r_[0:3, 60:68, 126:130, M // 2, M - 66:M])        # around the edges of tiles; all rows agree with 64-row tiles
    A = P.A64[rows]
    ref = A @ W
    bound = (2.0 ** -11 if act == "f16" else 2.0 ** -8) * np.abs(ref) + 256 * 2.0 ** -24 * (np.abs(A) @ np.abs(W)) + 2.0 ** -24
    assert bool((np.abs(to_f64(got)[rows] - ref) <= bound).all())


def test_second_launch():
    from paper_2504_12984_amd import binding as B
    gen = torch.Generator(device="cuda").manual_seed(62000)
    M, K, N, t = 1300, 8192, 16384, B.WType(B.QG_INT, 4)
    packed = torch.randint(0, 256, (K * N // 2,), dtype=torch.uint8, device="cuda", generator=gen)
    A = torch.randn(M, K, device="cuda", generator=gen).half()
    scales = (0.01 * torch.rand(K // 128, N, device="cuda", generator=gen)).half()
    got = B.qgemm(A, packed, scales, None, t, 128, N)
    B.qg_set_knob(2, 64)
    assert np.array_equal(bits_of(got), bits_of(B.qgemm(A, packed, scales, None, t, 128, N)))


@pytest.mark.parametrize("bits,zeros", [(4, "in"), (5, None), (8, "beyond")])
@pytest.mark.parametrize("N,M", [(16384, 257), (16448, 320), (16384, 600), (16448, 700), (16448, 1100), (16384, 1600)])
def test_mixed_heights_int8(N, M, bits, zeros):
    from paper_2504_12984_amd import binding as B
    gen = torch.Generator(device="cuda").manual_seed(63000 + M + bits)
    K, group = 256, (64, 128)[M % 3 == 0]
    t = B.WType(B.QG_INT if zeros is None else B.QG_UINT, bits)
    codes = torch.randint(0, 1 << bits, (K, N), dtype=torch.uint8, device="cuda", generator=gen)
    packed = B.repack(B.qg_pack_codes(codes, bits), t, K, N, layout=B.QG_LAYOUT_TILE128x64_I8)
    scales = (0.01 + 0.02 * torch.rand(K // group, N, device="cuda", generator=gen)).half()
    Z = None if zeros is None else torch.randint(0, 256 if zeros == "beyond" else 1 << bits, scales.shape, dtype=torch.uint8, device="cuda", generator=gen)
    A = torch.randint(-128, 128, (M, K), dtype=torch.int8, device="cuda", generator=gen)
    call = lambda: B.qgemm_a8(A, None, packed, scales, Z, t, group, N)      # noqa: E731
    B.qg_set_knob(0, 2)
    got = call()
    B.qg_set_knob(2, 64)
    assert np.array_equal(bits_of(got), bits_of(call()))
    rows = torch.tensor(sorted({0, 63, 64, 127, 128, M // 2, M - 65, M - 64, M - 1}))
    q = codes.cpu().double()
    q = q - (q >= 1 << (bits - 1)) * float(1 << bits) if zeros is None else q
    a, ref, size = A.cpu()[rows].double(), 0.0, 0.0
    for k in range(0, K, group):
        one = (a[:, k:k + group] @ (q[k:k + group] - (0 if Z is None else Z[k // group].cpu().double()))) * scales[k // group].cpu().double()
        ref, size = ref + one, size + one.abs()
    # integer sums of a group of at most 128 k are exact, groups are added in fp32
    bound = 2.0 ** -11 * ref.abs() + 2.0 ** -23 * (K // group + 2) * size + 2.0 ** -24
    assert bool(((got.cpu()[rows].double() - ref).abs() <= bound).all())
