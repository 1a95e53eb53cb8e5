"""Estimated duration of a chain's evaluation, by which the stamp sizes of a call
are placed on streams (compiled for the host from the library's header)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def cost(tmp_path_factory):
    d = tmp_path_factory.mktemp("cost")
    src = d / "cost.cpp"
    src.write_text('#include "bsi.h"\n#include "ctx.h"\n#include <cstdio>\nint main() {\n'
                   '  for (int n = 8; n <= 128; ++n)\n    for (int w = 1; w <= 4; ++w)\n'
                   '      std::printf("%d %d %.17g\\n", n, w, bsi_host::chain_cost(n, w));\n}\n')
    csrc = os.path.join(ROOT, "paper_2604_22048_amd", "csrc")
    subprocess.check_call(["hipcc", "-x", "c++", "-D__HIP_PLATFORM_AMD__", "-std=c++17", "-O0", "-I", csrc,
                           "-I", os.path.join(ROOT, "include"), "-I", "/opt/rocm/include", str(src), "-c", "-o",
                           str(d / "cost.o")])
    subprocess.check_call(["hipcc", str(d / "cost.o"), "-o", str(d / "cost")])
    out = subprocess.check_output([str(d / "cost")], text=True).split()
    return {(int(out[i]), int(out[i + 1])): float(out[i + 2]) for i in range(0, len(out), 3)}


def test_more_waves_shorten_a_chain_and_larger_sides_lengthen_it(cost):
    for n in range(8, 129):
        for w in (2, 3, 4):
            assert cost[n, w] < cost[n, w - 1]
        if n > 8:
            assert all(cost[n, w] > cost[n - 1, w] for w in (1, 2, 3, 4))


def test_only_the_pairs_are_shared(cost):
    """Twice the waves halve what grows with the side, not the rest."""
    fixed = 2 * cost[53, 2] - cost[53, 1]
    for n in (25, 53, 101):
        assert abs(2 * cost[n, 2] - cost[n, 1] - fixed) < 1e-6 and abs(4 * cost[n, 4] - cost[n, 1] - 3 * fixed) < 1e-6
    assert 0 < fixed < cost[101, 1]
