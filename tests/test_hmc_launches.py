"""Number of advance launches of a sampling call (the library's own rule,
called without a GPU): every iteration is run, whatever iters_per_launch."""
import ctypes as C

import pytest

INT_MAX = 2**31 - 1


@pytest.fixture(scope="module")
def launches():
    from paper_2604_22048_amd import _native
    f = _native.load()._ZN3bsi12hmc_launchesEiiibi
    f.restype, f.argtypes = C.c_int, [C.c_int, C.c_int, C.c_int, C.c_bool, C.c_int]
    return lambda T, ipl, L, nuts, depth=5: f(T, ipl, L, nuts, depth)


@pytest.mark.parametrize("nuts", [False, True])
@pytest.mark.parametrize("T", [1, 2, 40, 1300, 2**30, INT_MAX])
def test_all_in_one_launch(launches, T, nuts):
    for ipl in (T, INT_MAX - T + 1, INT_MAX - 1, INT_MAX):
        if ipl >= T:
            assert launches(T, ipl, 1, nuts) == 1


def test_short_launches_are_merged_and_long_ones_fit_an_int(launches):
    assert launches(0, 1, 20, False) == 0 and launches(0, INT_MAX, 20, True) == 0
    assert launches(40, 1, 20, False) == 2          # 25 trajectories of 20 steps
    assert launches(40, 7, 1000, False) == 6
    assert launches(40, 1, INT_MAX, False) == 40
    for T, L in ((1300, 20_000_000), (5000, 500_000)):
        n = launches(T, INT_MAX, L, False)
        assert -(-T // n) * L <= INT_MAX


@pytest.mark.parametrize("depth", range(1, 11))
def test_merged_nuts_launches_are_bounded(launches, depth):
    """Within twice 512 evaluations, however deep the trees, unless a launch is a
    single transition or asked for."""
    T = 200
    n = launches(T, 1, 20, True, depth)
    most = -(-T // n)
    assert most == 1 or most * 2**depth <= 1024
    assert n <= -(-T * 2**depth // 1024) and launches(T, 50, 20, True, depth) <= 4
