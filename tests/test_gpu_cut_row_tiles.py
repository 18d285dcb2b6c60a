"""Tiled kernel: 128-row tiles computed as two halves, for the types whose constants, unpack or LDS differ from the integers' (codebooks, floats, block
scales, groups of 32, the 16-bit pass-through), and in a second launch behind 256-row tiles.  That these shapes are cut so is
held in test_host_mixed_row_tiles.py.

An output's sums run over k in the same order whatever its tile, so they equal those of 64-row tiles bit for bit; the rows around the edges of
tiles are held against the oracle: |C - ref| <= u |ref| + K 2^-24 sum |a w| (fp32 sums), u = 2^-11 (fp16) or 2^-8 (bf16)."""
import numpy as np
import pytest
import torch

from paper_2504_12984_amd import workloads as WL
from gpu_util import Prepared, bits_of, to_f64
from test_gpu_codebook import CbCase
from test_gpu_mx import MxCase

pytestmark = pytest.mark.gpu
U, F, CB = WL.KIND_UINT, WL.KIND_FLOAT, WL.KIND_CODEBOOK


@pytest.fixture(autouse=True)
def _reset_knobs():
    yield
    from paper_2504_12984_amd import binding as B
    for k in range(4):
        B.qg_set_knob(k, 0)


# (path, kind, bits, exponent bits, mantissa bits, group, activations)
TYPES = {"codebook4": (2, CB, 4, 0, 0, 128, "f16"), "codebook8": (2, CB, 8, 0, 0, 128, "bf16"), "e3m2": (2, F, 6, 3, 2, 128, "f16"),
         "e2m2": (2, F, 5, 2, 2, 64, "bf16"), "mx_e2m1": (2, F, 4, 2, 1, 32, "bf16"), "mx_e4m3": (2, F, 8, 4, 3, 32, "bf16"),
         "u4_group32": (2, U, 4, 0, 0, 32, "f16"), "u8_group32": (2, U, 8, 0, 0, 32, "bf16"), "dense": (4, U, 5, 0, 0, 128, "f16")}


@pytest.mark.parametrize("M", [129, 961])
@pytest.mark.parametrize("name", TYPES)
def test_halves(name, M):
    from paper_2504_12984_amd import binding as B
    path, kind, bits, e, m, group, act = TYPES[name]
    K, N, mx = 256, 16448, name.startswith("mx")
    case = WL.Case(f"cut_{name}_{M}", M, K, N, kind, bits, e, m, group=group, act=act, scale_dtype="e8m0" if mx else "f16",
                   zero="random" if kind == U else None, seed=64000 + M + bits)
    P = (MxCase if mx else CbCase if kind == CB else Prepared)(case)
    B.qg_set_knob(0, path)
    got = P.gpu_c()
    B.qg_set_knob(2, 64)
    assert np.array_equal(bits_of(got), bits_of(P.gpu_c()))
    rows = np.unique(np.r_[0, 63:65, 127, M // 2, M - 66:M - 62, M - 1])
    A, W = to_f64(P.inp["A"])[rows], P.oracle_w()[0]
    ref = A @ W
    bound = (2.0 ** -11 if act == "f16" else 2.0 ** -8) * np.abs(ref) + K * 2.0 ** -24 * (np.abs(A) @ np.abs(W)) + 2.0 ** -24
    assert bool((np.abs(to_f64(got)[rows] - ref) <= bound).all())


def test_halves_in_a_second_launch():
    from paper_2504_12984_amd import binding as B
    gen = torch.Generator(device="cuda").manual_seed(65000)
    M, K, N, t = 769, 4096, 20480, B.WType(B.QG_INT, 4)
    packed = torch.randint(0, 256, (K * N // 2,), dtype=torch.uint8, device="cuda", generator=gen)
    A = torch.randn(M, K, device="cuda", generator=gen).half()
    scales = (0.01 * torch.rand(K // 128, N, device="cuda", generator=gen)).half()
    got = B.qgemm(A, packed, scales, None, t, 128, N)
    B.qg_set_knob(2, 64)
    assert np.array_equal(bits_of(got), bits_of(B.qgemm(A, packed, scales, None, t, 128, N)))
