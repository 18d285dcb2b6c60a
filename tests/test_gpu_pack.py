"""qg_pack_codes and repack against their bit-level definitions, at the edges of their tiles:
counts around a workgroup's 8192 codes, buffers that start at odd addresses, strips that do not
fill a workgroup, every code width and every arrangement of a lane's codes."""
import numpy as np
import pytest
import torch

from oracle import qgemm_oracle as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits", range(1, 9))
def test_pack_counts_and_odd_addresses(bits):
    from paper_2504_12984_amd import binding as B
    rng = np.random.default_rng(bits)
    buf = torch.from_numpy(rng.integers(0, 256, 3 * 8192 + 64, dtype=np.uint8)).cuda()      # bits above the code are ignored
    for count in (1, 7, 8, 31, 33, 8191, 8192, 8193, 2 * 8192, 3 * 8192 - 5):
        for start in (0, 1, 6):
            view = buf[start:start + count]
            got = B.qg_pack_codes(view, bits).cpu().numpy()
            want = O.pack_canonical(view.cpu().numpy() & ((1 << bits) - 1), bits)
            assert np.array_equal(got, want), (bits, count, start)


def _place(codes, bits, mode, flip):
    """The device layout from its definition: one row of bytes per chunk, bit by bit."""
    K, N = codes.shape
    lane, t = np.meshgrid(np.arange(64), np.arange(32 if mode == "i8" else 64), indexing="ij")
    if mode == "i8":
        parts = [(64 * (t // 16) + 16 * (lane // 16) + 4 * (t & 3) + e, 4 * (lane % 16) + ((t >> 2) & 3), 8, e) for e in range(4)]
    elif mode.startswith("r32"):
        parts = [(16 * (t // 8) + 8 * (lane // 32) + 2 * (t & 3) + h, 2 * (lane % 32) + ((t >> 2) & 1), 16, h) for h in range(2)]
    else:
        parts = [(32 * (t // 16) + 8 * (lane // 16) + 2 * (t & 3) + h, 4 * (lane % 16) + ((t >> 2) & 3), 16, h) for h in range(2)]
    out = []
    for nc in range(N // 64):
        for kc in range(K // 128):
            tile = codes[128 * kc:128 * kc + 128, 64 * nc:64 * nc + 64] ^ flip
            words = np.zeros((64, 4 * bits), dtype=np.uint32)
            for k, n, width, part in parts:
                for j in range(bits):
                    if mode.endswith("plain"):
                        pos = (2 * t + part) * bits + j
                        reg, at = pos // 32, pos % 32
                    else:
                        pos = t * bits + j
                        reg, at = pos // width, pos % width + width * part
                    np.bitwise_or.at(words, (lane, reg), (((tile[k, n] >> j) & 1).astype(np.uint32)) << at.astype(np.uint32))
            out.append(words.reshape(64, bits, 4).transpose(1, 0, 2).copy().view(np.uint8).reshape(-1))
    return np.concatenate(out)


@pytest.mark.parametrize("mode", ["streams", "plain", "r32", "r32_plain", "i8"])
@pytest.mark.parametrize("bits", range(1, 9))
def test_repack_every_arrangement(bits, mode):
    from paper_2504_12984_amd import binding as B
    rng = np.random.default_rng(10 * bits + len(mode))
    layout = {"i8": B.QG_LAYOUT_TILE128x64_I8, "r32": B.QG_LAYOUT_TILE128x64_R32,
              "r32_plain": B.QG_LAYOUT_TILE128x64_R32}.get(mode, B.QG_LAYOUT_TILE128x64)
    flip = 0
    if mode == "plain":
        wt = B.WType(B.QG_CODEBOOK, bits)
    elif mode == "r32_plain":
        split = {4: (2, 1), 6: (3, 2), 8: (4, 3)}
        if bits not in split:
            pytest.skip("no type of this width in plain order on the second layout")
        wt = B.WType(B.QG_FLOAT, bits, *split[bits])
    else:
        signed = bits % 2 == 1
        wt = B.WType(B.QG_INT if signed else B.QG_UINT, bits)
        flip = 1 << (bits - 1) if signed else 0
    for K, N in ((128, 64), (256, 320), (384, 576)):
        codes = rng.integers(0, 1 << bits, (K, N), dtype=np.uint8)
        stream = torch.from_numpy(np.concatenate([np.zeros(3, np.uint8), O.pack_canonical(codes, bits)])).cuda()
        for off in (0, 3):                    # a stream that starts at an odd address
            s = stream[3:] if off else stream[3:].clone()
            got = B.repack(s, wt, K, N, layout=layout).cpu().numpy()
            assert np.array_equal(got, _place(codes, bits, mode, flip)), (bits, mode, K, N, off)
