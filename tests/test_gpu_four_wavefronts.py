"""Several row tiles on four wavefronts, one strip or two per workgroup, against the oracle: rows at the tiles' edges, wavefronts with
no chunk, one and several, K whole and in slabs."""
import pytest

from paper_2504_12984_amd import workloads as WL
from gpu_util import Prepared, assert_c_close

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _reset_knobs():
    yield
    from paper_2504_12984_amd import binding as B
    for k in range(4):
        B.qg_set_knob(k, 0)


def _case(name, M, K, N, i, kind=WL.KIND_UINT, bits=4, group=128):
    zero = {"zero": "random", "zero_hi": (1 << bits) - 1} if kind == WL.KIND_UINT else {}
    return Prepared(WL.Case(name, M, K, N, kind, bits, group=group, act="bf16" if i % 2 else "f16", scale_dtype="f16", seed=55000 + i, **zero))


@pytest.mark.parametrize("variant,M", [(22, 17), (22, 24), (22, 32), (27, 18), (27, 31), (32, 33), (37, 48), (42, 49), (47, 64)])
@pytest.mark.parametrize("K,bits,group", [(256, 4, 128), (1024, 8, 64), (1408, 3, 128), (3712, 5, 64)])
def test_arrangements(variant, M, K, bits, group):
    from paper_2504_12984_amd import binding as B
    P = _case(f"four_{variant}_{M}_{K}", M, K, 512, variant + M, bits=bits, group=group)
    C = P.oracle_c()
    B.qg_set_knob(3, variant)
    for splitk in (1, 3):
        B.qg_set_knob(1, min(splitk, K // 256))
        assert_c_close(P.gpu_c(), C, f"{P.case.name} {splitk}")


@pytest.mark.parametrize("M,K,N,bits,group", [(20, 512, 33472, 4, 128), (17, 1024, 4096, 4, 32), (24, 1024, 16384, 8, 64), (18, 4096, 8256, 4, 128),
                                              (32, 1024, 33408, 6, 128), (20, 512, 24576, 3, 64),
                                              (33, 1024, 2048, 4, 128), (48, 512, 24576, 4, 64), (64, 2048, 2048, 8, 128), (49, 512, 18432, 8, 64),
                                              (45, 1408, 512, 6, 32), (63, 1024, 320, 8, 32)])
def test_automatic_choice(M, K, N, bits, group):
    from paper_2504_12984_amd import binding as B
    P = _case(f"four_auto_{M}_{K}_{N}", M, K, N, M + bits, bits=bits, group=group)
    assert B.qg_plan(P.wtype, group, M, N, K)["variant"] in (22, 27, 32, 37, 42, 47)
    assert_c_close(P.gpu_c(), P.oracle_c(), P.case.name)


@pytest.mark.parametrize("bits,ebits,mbits,act", [(6, 3, 2, "f16"), (8, 4, 3, "bf16")])
def test_wide_floats_on_four_row_tiles(bits, ebits, mbits, act):
    from paper_2504_12984_amd import binding as B
    P = Prepared(WL.Case(f"four_f{bits}", 63, 2176, 512, WL.KIND_FLOAT, bits, ebits, mbits, group=128, act=act, scale_dtype="f16", zero=None, seed=55100 + bits))
    assert B.qg_plan(P.wtype, 128, 63, 512, 2176)["variant"] == 42
    assert_c_close(P.gpu_c(), P.oracle_c(), P.case.name)
