"""33 to 48 rows on three 16-row tiles of the streaming kernel (arrangements 31 and 36): the same
chunks per wavefront and the same order of sums as with four row tiles (41, 46, checked against the oracle
elsewhere), so the results are the same bits; one case each against the oracle."""
import numpy as np
import pytest
import torch

from paper_2504_12984_amd import workloads as WL
from gpu_util import Prepared, assert_c_close, bits_of

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _reset_knobs():
    yield
    from paper_2504_12984_amd import binding as B
    for k in range(4):
        B.qg_set_knob(k, 0)


@pytest.mark.parametrize("M", [33, 47, 48])
@pytest.mark.parametrize("kind,bits,group,act,scale", [
    ("u", 4, 128, "f16", "f16"), ("i", 3, 64, "bf16", "bf16"), ("u", 8, 0, "bf16", "f16"), ("u", 5, 32, "f16", "f16"),
    ("f", 6, 128, "bf16", "f16"), ("f", 4, 32, "bf16", "e8m0"), ("f", 8, 32, "f16", "e8m0"), ("cb", 4, 64, "f16", "f16")])
def test_three_row_tiles_give_the_bits_of_four(M, kind, bits, group, act, scale):
    from paper_2504_12984_amd import binding as B
    K, N = 1408, 512
    gen = torch.Generator(device="cuda").manual_seed(100 * M + bits)
    t = {"u": B.WType(B.QG_UINT, bits), "i": B.WType(B.QG_INT, bits), "cb": B.WType(B.QG_CODEBOOK, bits)}.get(kind)
    if t is None:
        t = B.WType(B.QG_FLOAT, bits, *{4: (2, 1), 6: (3, 2), 8: (4, 3)}[bits])
    dt = torch.float16 if act == "f16" else torch.bfloat16
    codes = torch.randint(0, (1 << bits) - 1, (K, N), dtype=torch.uint8, device="cuda", generator=gen)
    codes = torch.where((codes & 0x7F) == 0x7F, codes ^ 1, codes) if (kind, bits) == ("f", 8) else codes
    packed = B.repack(B.qg_pack_codes(codes, bits), t, K, N)
    rows = K // group if group else 1
    if scale == "e8m0":
        S = torch.randint(117, 125, (rows, N), dtype=torch.uint8, device="cuda", generator=gen)
    else:
        S = (0.01 + 0.02 * torch.rand(rows, N, device="cuda", generator=gen)).to(torch.float16 if scale == "f16" else torch.bfloat16)
    Z = torch.randint(0, 1 << bits, (rows, N), dtype=torch.uint8, device="cuda", generator=gen) if kind == "u" else None
    A = torch.randn(M, K, device="cuda", generator=gen).to(dt)
    levels = torch.randn(1 << bits, device="cuda", generator=gen).half()
    arrangements = [(31, 41)] if group == 32 and scale != "e8m0" else [(31, 41), (36, 46)]
    for three, four in arrangements:
        for splitk in (1, 3):
            got = []
            for variant in (three, four, three):
                B.qg_set_knob(1, splitk)
                B.qg_set_knob(3, variant)
                C = B.qgemm_codebook(A, packed, levels, S, bits, group, N) if kind == "cb" else B.qgemm(A, packed, S, Z, t, group, N)
                got.append(bits_of(C))
            assert np.array_equal(got[0], got[1]) and np.array_equal(got[0], got[2]), (three, splitk)


@pytest.mark.parametrize("M,N", [(33, 128), (40, 6144), (48, 320)])
def test_automatic_choice_against_the_oracle(M, N):
    P = Prepared(WL.Case(f"three_{M}_{N}", M, 4096, N, WL.KIND_UINT, 4, group=64, zero=7, seed=53000 + M))
    assert_c_close(P.gpu_c(), P.oracle_c(), P.case.name)
