"""LDS of the forward DFT's workgroups (the library's own sizes, without a GPU):
every operand read of the two passes, the steps read ahead past the operands'
end included, lies within what the launch allocates."""
import ctypes as C
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2604_22048_amd", "csrc")
PLANS = (1, 2, 3, 4, 5, 6, 8)


@pytest.fixture(scope="module")
def lds_bytes():
    from paper_2604_22048_amd import _native
    f = _native.load()._ZN3bsi23dft_bins_mfma_lds_bytesEii
    f.restype, f.argtypes = C.c_size_t, [C.c_int, C.c_int]
    return f


def _ahead():
    with open(os.path.join(CSRC, "dft_device.h")) as f:
        return int(re.search(r"constexpr int kAhead = (\d+);", f.read()).group(1))


@pytest.mark.parametrize("N", range(8, 129))
def test_operand_reads_stay_inside(lds_bytes, N):
    ahead, steps, nrow = _ahead(), (N + 3) // 4, N // 2 + 1
    last = max(ahead, steps // ahead * ahead + ahead) - 1      # the last step whose operands are loaded
    col = 16 * ((N + 15) // 16) - 1                            # the last column of a block
    stamp_end = 4 * ((4 * last + 3) * N + col + 1)             # pass A: float rows of N
    ld = 4 * steps + (0 if steps % 2 else 4)
    q_end = 8 * ((nrow - 1) * ld + 4 * last + 3 + 1)           # pass B: complex rows of ld
    for P in PLANS:
        if 64 * P // ((N - (N + 1) % 2 - 1) // 2 + 1) < 1:
            continue
        assert max(stamp_end, q_end) <= lds_bytes(N, P) <= 160 * 1024 - 64, P
