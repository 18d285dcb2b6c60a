"""Host logic: where several row tiles take four wavefronts instead of eight (qg_plan; the times stand at the rule)."""
import pytest

from paper_2504_12984_amd import binding as B

U = {bits: B.WType(B.QG_UINT, bits) for bits in (1, 2, 4, 6, 7, 8)}
CB = {bits: B.WType(B.QG_CODEBOOK, bits) for bits in (4, 5, 8)}
F4, F6 = B.WType(B.QG_FLOAT, 4, 2, 1), B.WType(B.QG_FLOAT, 6, 3, 2)
F7, F8 = B.WType(B.QG_FLOAT, 7, 3, 3), B.WType(B.QG_FLOAT, 8, 4, 3)


@pytest.mark.parametrize("t,M,K,N,variant,splitk", [
    (U[4], 21, 1024, 57152, 22, 1), (U[4], 20, 2048, 57344, 27, 1), (CB[5], 32, 512, 34304, 27, 1),      # several rounds of workgroups
    (U[4], 20, 8192, 24640, 22, 1), (U[4], 32, 8192, 24640, 21, 1), (CB[4], 28, 8192, 24640, 22, 1),     # a round and a fraction
    (U[4], 20, 8192, 10240, 22, 2), (U[4], 20, 8192, 12224, 22, 2), (U[4], 32, 8192, 10240, 21, 2),
    (U[4], 20, 8192, 8192, 21, 2), (U[4], 20, 8192, 12288, 21, 1),
    (U[4], 20, 1024, 4096, 22, 1), (U[4], 28, 1024, 4096, 21, 1), (U[8], 28, 1024, 4096, 22, 1), (CB[8], 20, 1024, 4096, 21, 1),      # two chunks each
    (U[4], 20, 512, 28672, 27, 1), (U[8], 20, 1408, 28672, 27, 1), (U[4], 24, 4096, 28672, 26, 1), (F6, 20, 1408, 28672, 26, 1)])
def test_two_row_tiles(t, M, K, N, variant, splitk):
    p = B.qg_plan(t, 128, M, N, K)
    assert (p["path"], p["variant"], p["splitk"]) == (1, variant, splitk), p


def test_two_row_tiles_groups_of_32():
    # no pairs of strips there: from 257 strips on a round and a fraction whatever their number
    assert B.qg_plan(U[4], 32, 24, 28672, 1024)["variant"] == 22
    assert B.qg_plan(U[4], 32, 32, 28672, 8192)["variant"] == 21
    assert B.qg_plan(F4, 32, 20, 57344, 1024, act=B.QG_BF16, scale_dtype=B.QG_E8M0)["variant"] == 27


@pytest.mark.parametrize("t,group,M,K,N,variant", [
    (U[8], 128, 64, 2048, 2048, 42), (U[8], 64, 49, 512, 18432, 47), (U[6], 128, 64, 8192, 4096, 41),      # registers
    (U[7], 128, 64, 8192, 4096, 42), (U[6], 64, 64, 8192, 4096, 42), (U[7], 128, 48, 8192, 4096, 31), (F8, 128, 64, 8192, 4096, 42), (F6, 128, 49, 2048, 8192, 42), (F7, 128, 64, 8192, 4096, 41),
    (U[6], 32, 40, 4096, 2048, 32), (U[8], 32, 64, 1024, 8192, 42), (U[4], 32, 64, 4096, 2048, 41),
    (U[4], 128, 33, 1024, 8192, 32), (U[4], 128, 33, 768, 8192, 31), (CB[4], 128, 40, 1024, 8192, 31), (CB[8], 128, 52, 1024, 16384, 42),      # two chunks each
    (U[8], 128, 33, 512, 24640, 32), (CB[4], 128, 40, 512, 24640, 32), (CB[4], 128, 52, 512, 24640, 41), (F6, 128, 40, 2048, 16384, 32),      # a round and a fraction, all CUs
    (F6, 128, 40, 512, 28672, 37), (CB[8], 128, 52, 1024, 16512, 47), (F6, 128, 40, 512, 18432, 36)])                     # pairs of strips
def test_three_and_four_row_tiles(t, group, M, K, N, variant):
    p = B.qg_plan(t, group, M, N, K)
    assert (p["path"], p["variant"]) == (1, variant), p
