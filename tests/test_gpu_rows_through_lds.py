"""From 13 or 16 rows on the streaming kernels bring A to the matrix instruction through LDS, with fewer they load it as the
instruction reads it.  Chunks per wavefront and the order of the sums are the same, so a row's results are the
same bits whichever way it came; one case per arrangement against the oracle."""
import numpy as np
import pytest
import torch

from paper_2504_12984_amd import workloads as WL
from gpu_util import Prepared, assert_c_close, bits_of

pytestmark = pytest.mark.gpu
K, N = 1408, 512                 # eleven chunks: wavefronts with none, one and two


@pytest.fixture(autouse=True)
def _reset_knobs():
    yield
    from paper_2504_12984_amd import binding as B
    for k in range(4):
        B.qg_set_knob(k, 0)


def _weight(kind, bits, rows, gen):
    from paper_2504_12984_amd import binding as B
    t = {"u": B.WType(B.QG_UINT, bits), "cb": B.WType(B.QG_CODEBOOK, bits)}.get(kind) or B.WType(B.QG_FLOAT, bits, *{4: (2, 1), 6: (3, 2)}[bits])
    codes = torch.randint(0, 1 << bits, (K, N), dtype=torch.uint8, device="cuda", generator=gen)
    scales = (0.01 + 0.02 * torch.rand(rows, N, device="cuda", generator=gen)).half()
    return t, codes, scales


@pytest.mark.parametrize("variant", [10, 11, 12, 14, 15, 16])
@pytest.mark.parametrize("kind,bits,group", [("u", 4, 128), ("u", 8, 64), ("f", 6, 0), ("f", 4, 32), ("cb", 3, 128), ("cb", 8, 64)])
def test_a_row_has_the_same_bits_either_way(kind, bits, group, variant):
    from paper_2504_12984_amd import binding as B
    gen = torch.Generator(device="cuda").manual_seed(10 * variant + bits)
    t, codes, scales = _weight(kind, bits, K // group if group else 1, gen)
    mx = (kind, group) == ("f", 32)                                    # block scales
    if mx:
        scales = torch.randint(117, 125, scales.shape, dtype=torch.uint8, device="cuda", generator=gen)
    packed = B.repack(B.qg_pack_codes(codes, bits), t, K, N)
    act = torch.bfloat16 if variant % 2 else torch.float16
    A = torch.randn(16, K, device="cuda", generator=gen).to(act)
    levels = torch.randn(1 << bits, device="cuda", generator=gen).half()
    B.qg_set_knob(3, variant)
    got = {}
    for M in (1, 12, 13, 15, 16):
        B.qg_set_knob(1, 2 if M in (12, 13, 16) else 1)
        C = B.qgemm_codebook(A[:M], packed, levels, scales, bits, group, N) if kind == "cb" else B.qgemm(A[:M], packed, scales, None, t, group, N)
        got[M] = bits_of(C)
    assert np.array_equal(got[13][:12], got[12]) and np.array_equal(got[16][:13], got[13])
    assert np.array_equal(got[15][:1], got[1])


@pytest.mark.parametrize("variant,M", [(10, 13), (12, 16), (16, 15), (21, 17), (26, 31), (31, 33), (36, 48), (41, 49), (46, 64)])
def test_arrangements_against_the_oracle(variant, M):
    from paper_2504_12984_amd import binding as B
    P = Prepared(WL.Case(f"lds_{variant}_{M}", M, K, N, WL.KIND_UINT, 3 + variant % 4, group=(64, 128, K)[M % 3], zero="random", zero_hi=7,
                         act="bf16" if M % 2 else "f16", scale_dtype="f16", seed=54000 + variant))
    for splitk in (1, 3):
        B.qg_set_knob(1, splitk)
        B.qg_set_knob(3, variant)
        assert_c_close(P.gpu_c(), P.oracle_c(), f"{P.case.name} {splitk}")


@pytest.mark.parametrize("variant,M,workgroups", [
    (14, 16, 5), (14, 3, 9), (15, 13, 13), (15, 16, 9), (16, 16, 5), (16, 1, 13), (26, 20, 13), (26, 32, 9), (36, 40, 5), (46, 64, 9),
    (10, 16, 5), (12, 16, 3), (21, 27, 5), (31, 33, 5), (41, 64, 5)])
def test_long_k_whole(variant, M, workgroups):
    """More chunks than a wavefront has in flight, an odd number of them (41): every chunk's rows pass through the same part of
    LDS.  Several strips per workgroup, K longer than 32 chunks: strips dealt to XCDs in runs, workgroup counts that eight does not divide."""
    from paper_2504_12984_amd import binding as B
    strips = {14: 2, 15: 2, 16: 4, 26: 2, 36: 2, 46: 2}.get(variant, 1)
    P = Prepared(WL.Case(f"long_{variant}_{M}", M, 128 * 41, 64 * strips * workgroups, WL.KIND_UINT, 4 if variant % 2 else 3, group=64 if M % 3 == 0 else 128,
                         zero="random", zero_hi=7, act="bf16" if M % 2 else "f16", scale_dtype="f16", seed=54100 + variant + M))
    B.qg_set_knob(1, 1)
    B.qg_set_knob(3, variant)
    assert_c_close(P.gpu_c(), P.oracle_c(), P.case.name)
