"""Host logic: tile height and split-K of 16-bit calls with more than 64 rows where slabs meet in the kernel (qg_plan; the times stand at
the estimate)."""
import pytest

from paper_2504_12984_amd import binding as B

U4, I2, CB8 = B.WType(B.QG_UINT, 4), B.WType(B.QG_INT, 2), B.WType(B.QG_CODEBOOK, 8)


@pytest.mark.parametrize("t,group,M,K,N,tile,splitk", [
    (U4, 128, 112, 3072, 11008, 64, 2), (U4, 64, 409, 1536, 2880, 64, 1), (U4, 128, 929, 2304, 2112, 64, 1), (I2, 32, 93, 2944, 11072, 128, 4),
    (U4, 128, 300, 8192, 8192, 128, 2), (U4, 128, 300, 4096, 4096, 64, 3), (U4, 128, 200, 5120, 13824, 128, 2), (CB8, 128, 128, 4096, 14336, 128, 4)])
def test_slabs_that_meet_in_the_kernel(t, group, M, K, N, tile, splitk):
    p = B.qg_plan(t, group, M, N, K)
    assert (p["path"], p["row_tile"], p["splitk"]) == (2, tile, splitk), p

