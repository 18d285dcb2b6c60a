"""Which of the streaming kernel's ways of A a call of one row tile takes (the last template argument of the kernel it launches)."""
import pytest

from test_host_workspace import _run, stub  # noqa: F401


@pytest.mark.parametrize("M,K,N,bits,group,through_lds", [
    (16, 4096, 8192, 4, 128, False), (16, 2048, 16384, 6, 128, False), (16, 4096, 8192, 8, 128, True),        # two chunks for each of eight wavefronts
    (16, 8192, 14336, 4, 128, True), (15, 8192, 14336, 4, 128, False),                                        # four
    (16, 1024, 28672, 3, 64, False), (16, 512, 28672, 3, 64, True), (13, 2048, 28672, 4, 64, True),           # two strips: two, one, four
    (16, 2048, 57344, 4, 128, True), (13, 2048, 57344, 4, 128, False),                                        # four strips
    (16, 1024, 4096, 4, 32, False), (13, 2048, 16384, 4, 32, True)])                                          # groups of 32, four wavefronts: two, four
def test_way_of_a(stub, M, K, N, bits, group, through_lds):  # noqa: F811
    (c,) = _run(stub, f"out = [linear({M}, {K}, {N}, {bits}, {group})]")
    names = [n for k, n, *_ in c["launches"] if k == "decode_kernel"]
    assert len(names) == 1 and names[0].split("EEEv")[0].endswith(f"Lb{int(through_lds)}"), c["launches"]
