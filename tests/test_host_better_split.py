"""Host logic: slabs of the streaming kernel where the strips are no power of two (qg_plan; the times stand at the rule)."""
import pytest

from paper_2504_12984_amd import binding as B
from test_host_workspace import _run, stub  # noqa: F401

U4, U8, I2, F6 = B.WType(B.QG_UINT, 4), B.WType(B.QG_UINT, 8), B.WType(B.QG_INT, 2), B.WType(B.QG_FLOAT, 6, 3, 2)


@pytest.mark.parametrize("t,M,K,N,splitk", [
    (U4, 1, 13824, 5120, 3), (U4, 16, 13824, 5120, 3), (U4, 32, 13824, 5120, 3), (U4, 48, 13824, 5120, 3),      # 80 strips: 240 workgroups
    (U8, 16, 8192, 7168, 2), (U8, 1, 16384, 3072, 5),
    (U4, 32, 4096, 10240, 1), (U4, 48, 4096, 10240, 1), (I2, 64, 4096, 10240, 1),      # 160 strips: whole, not two rounds of halves
    (U4, 16, 8192, 8192, 2), (U4, 32, 8192, 8192, 2), (U4, 16, 14336, 4096, 4), (U4, 16, 4096, 14336, 1),      # as before
    (F6, 1, 8192, 7168, 2), (U4, 20, 13824, 5120, 4), (U4, 32, 8192, 10240, 2)])      # where the estimate does not hold
def test_slabs(t, M, K, N, splitk):
    p = B.qg_plan(t, 128, M, N, K)
    assert (p["path"], p["splitk"]) == (1, splitk), p


@pytest.mark.parametrize("M", [1, 16, 28, 40, 64])
@pytest.mark.parametrize("K", [512, 2560, 4096, 5120, 13824, 16384])
def test_slabs_invariants(M, K):
    for t in (U4, U8, I2, F6):
        for strips in range(1, 256, 3):
            B.qg_set_knob(0, 1)
            p = B.qg_plan(t, 128, M, 64 * strips, K)
            B.qg_set_knob(0, 0)
            sk, cps, KC = p["splitk"], p["chunks_per_slab"], K // 128
            assert 1 <= sk <= 8 and sk * cps >= KC > (sk - 1) * cps          # slabs cover K, none is empty
            row_tiles = p["variant"] // 10
            assert sk == 1 or (strips * sk < 512 and 4096 * row_tiles * strips * sk <= 32 << 20)          # the workspace's capacity
            assert sk == 1 or row_tiles > 2 or 4096 * row_tiles * strips * (sk - 1) <= 4 << 20          # and that of the slots


def test_slabs_int8(stub):
    # a launch has strips x slabs workgroups: whole rather than two rounds of halves, three slabs of 80 strips rather than four
    shapes = [(16, 4096, 14336, 1), (64, 4096, 10240, 1), (16, 13824, 5120, 3), (64, 5120, 5120, 3), (16, 8192, 8192, 2)]
    calls = _run(stub, "out = [" + ", ".join(f"a8({M}, {K}, {N})" for M, K, N, _ in shapes) + "]")
    for (M, K, N, slabs), c in zip(shapes, calls):
        assert c["rc"] == 0 and c["launches"][-1][0] == "a8_kernel" and c["launches"][-1][2:] == [N // 64, slabs], (M, K, N, c)
