"""Estimated duration of an evaluation, by which a call's stamp sizes are placed on
streams (the library's own rule, called without a GPU), against durations
measured on the device."""
import ctypes as C

import pytest


@pytest.fixture(scope="module")
def us():
    from paper_2604_22048_amd import _native
    f = _native.load()._ZN3bsi11hmc_eval_usEiiiiNS_8EvalFormE
    f.restype, f.argtypes = C.c_double, [C.c_int] * 5
    return lambda N, chains=2, n_exp=1, wpc=1, form=0: f(N, chains, n_exp, wpc, form)


GENERAL, FIXED, TEAM = 0, 1, 2
# us of one galaxy's evaluation: (side, chains, exposures, form)
MEASURED = {(8, 2, 1, GENERAL): 1.95, (16, 2, 1, GENERAL): 1.93, (30, 2, 1, GENERAL): 1.71, (48, 2, 1, GENERAL): 2.79,
            (64, 2, 1, GENERAL): 4.07, (80, 2, 1, GENERAL): 5.35, (90, 2, 1, GENERAL): 6.04,
            (115, 2, 1, GENERAL): 7.00, (127, 2, 1, GENERAL): 7.63, (16, 6, 1, GENERAL): 2.34,
            (64, 6, 1, GENERAL): 5.08, (101, 6, 1, GENERAL): 7.42, (127, 8, 1, GENERAL): 10.21,
            (48, 2, 2, GENERAL): 5.31, (80, 2, 2, GENERAL): 10.61, (53, 1, 1, FIXED): 2.55, (73, 1, 1, FIXED): 3.55,
            (101, 1, 1, FIXED): 5.25, (25, 1, 1, FIXED): 1.03, (25, 2, 1, TEAM): 1.26, (53, 1, 1, TEAM): 1.43, (73, 2, 1, TEAM): 1.78,
            (101, 2, 1, TEAM): 2.19}


@pytest.mark.parametrize("case", MEASURED)
def test_estimate_is_near_what_was_measured(us, case):
    """To 25 %: enough that of two sides whose durations differ by more than half,
    the longer one is taken for it."""
    N, chains, n_exp, form = case
    assert 0.75 < us(N, chains, n_exp, 1, form) / MEASURED[case] < 1.25


SPLIT = {(41, 2): 1.56, (53, 2): 1.73, (73, 2): 2.65, (101, 2): 4.1, (41, 4): 1.65, (53, 4): 1.81, (73, 4): 2.10,
         (101, 4): 2.91}


@pytest.mark.parametrize("N,waves", SPLIT)
def test_estimate_of_chains_over_several_waves(us, N, waves):
    """The waves share a chain's pairs, not what each of them repeats."""
    assert 0.75 < us(N, 1, 1, waves, FIXED) / SPLIT[N, waves] < 1.25


def test_order(us):
    for chains in (1, 4, 8):
        assert all(us(n + 1, chains) >= us(n, chains) for n in range(8, 128))
    assert us(127) > 3 * us(8) and us(101, form=TEAM) < us(101, form=FIXED) < us(101) and us(127, 8) > us(127, 4)
    for w in (2, 4):
        assert us(101, 1, 1, w) < us(101, 1, 1, w // 2) and us(101, 1, 2, w) > us(101, 1, 1, w)
