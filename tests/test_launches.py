"""Which kernels a call launches, and with which operands it calls rocBLAS: the library's host code on stand-ins for the HIP runtime
(launches.py).  No GPU."""
import pytest

import launches


@pytest.fixture(scope="module")
def recorded(tmp_path_factory):
    so = launches.build(str(tmp_path_factory.mktemp("launches")))
    return lambda script: launches.record(so, script)


# bf16 splits into two factors that are no chunk of the chunk kernels, whose passes hold the spectrum of k in fp32, go to the kernel that
# is fp32 throughout, at any number of rows
def test_splits_whose_kernel_spectrum_is_fp32(recorded):
    got = recorded("""
result = []
for factors in [(16, 32), (32, 16), (16, 64), (64, 16), (16, 128), (128, 16), (32, 128), (128, 32)]:
    nfft = factors[0] * factors[1]
    for B, H in [(1, 1), (1, 4096), (2, 3), (5, 768), (2, 3072), (8, 1536)]:
        for n, klen in [(nfft // 2, nfft // 2), (40, 40), (41, 9), (nfft, nfft)]:
            result.append(calls.conv(B, H, n, klen, factors))
""")
    for kernels in got:
        assert len(kernels) == 1 and kernels[0].startswith("conv_kernel "), kernels
