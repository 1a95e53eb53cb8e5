"""Waves that a launch's chain groups count for, and whether they are evaluated by
teams (the library's own rules, called without a GPU through a host program):
teams exist for the specialised sides on their default plans only."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2604_22048_amd")
SPECIALISED = (25, 41, 53, 73, 101)

PROGRAM = r"""
#include <cstdio>
#include "bsi_kernels.h"
#include "kspace.h"
int main() {
  for (int n = 8; n <= 128; ++n)
    for (int C = 1; C <= 8; ++C)
      for (int nuts = 0; nuts < 2; ++nuts)
        for (int prof = 0; prof < 3; ++prof) {
          bsi::HmcArgs a{};
          a.N = n;
          a.P = bsi::make_slot_plan(n).P;
          a.C = C;
          a.prof = prof;
          a.nuts = nuts;
          a.wpc = 1;
          a.n_gal = 2;
          std::printf("%d %d %d %d %lld %d\n", n, C, nuts, prof, (long long)bsi::hmc_team_waves(a), (int)bsi::hmc_runs_teams(a));
        }
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    from paper_2604_22048_amd import _native, build
    _native.load()
    d = tmp_path_factory.mktemp("rules")
    (d / "rules.cpp").write_text(PROGRAM)
    subprocess.check_call([build.HIPCC, "-x", "hip", "--offload-host-only", "-std=c++17", "-O0", "-I",
                           os.path.join(PKG, "csrc"), "-I", os.path.join(ROOT, "include"), str(d / "rules.cpp"), "-x", "none",
                           _native.LIB_PATH, "-Wl,-rpath," + PKG, "-o", str(d / "rules")])
    out = subprocess.check_output([str(d / "rules")], text=True).split()
    rows = [tuple(int(x) for x in out[i:i + 6]) for i in range(0, len(out), 6)]
    return {r[:4]: r[4:] for r in rows}


def test_other_sides_count_one_wave_a_chain(rules):
    for (n, chains, nuts, prof), (waves, teams) in rules.items():
        if n not in SPECIALISED or chains > 4 or prof == 1:
            assert waves == 2 * chains and not teams, (n, chains, nuts, prof)


def test_specialised_sides_count_their_teams(rules):
    for n in SPECIALISED:
        for prof in (0, 2):
            waves, teams = rules[n, 4, 0, prof]
            assert teams and waves >= 4, n
            assert rules[n, 4, 1, prof][1] == (n >= 53), n
    assert not rules[25, 1, 0, 0][1] and rules[53, 1, 0, 0][1]
