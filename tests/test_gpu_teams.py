"""Trajectories by teams of waves: a few galaxies, whose chain groups are each
evaluated by several waves, draw the same samples, to the last bit, as the same
galaxies among so many that one wave evaluates each group."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from workloads import gen              # noqa: E402
from tests import synth                # noqa: E402

MANY = 1100        # beyond the 1,024 groups of the largest line


@pytest.fixture(scope="module")
def bsi(device):
    from paper_2604_22048_amd import api
    return api


# (side, chains, profile, warmup, draws, leapfrog steps or "nuts", jitter): every
# team kernel, one step a trajectory, several launches, an odd number of chains
FORMS = [(25, 1), (25, 2), (25, 4), (41, 2), (41, 4), (53, 1), (53, 2), (53, 4), (73, 1), (101, 1)]
CASES = [(N, C, p, 5, 9, 7, 0.1) for N, C in FORMS for p in ("exp", "spergel")]
CASES += [(N, C, p, 5, 9, "nuts", 0.0) for N, C in FORMS if N != 41 or C != 2 for p in ("exp", "spergel")]
CASES += [(53, 1, "exp", 3, 4, 1, 0.1), (53, 4, "exp", 10, 20, 20, 0.1), (73, 3, "exp", 3, 4, 5, 0.0),
          (101, 4, "exp", 3, 4, 5, 0.1), (73, 4, "exp", 3, 40, "nuts", 0.0), (53, 8, "exp", 3, 4, 5, 0.1),
          (73, 5, "exp", 3, 4, "nuts", 0.0)]


@pytest.mark.parametrize("N,C,profile,warmup,draws,L,jitter", CASES)
def test_team_draws_are_one_waves(bsi, N, C, profile, warmup, draws, L, jitter):
    import torch
    t, params, data, off = synth.make_population("uneven", n_gal=2, seed=N + C, sizes=[N] * 2)
    init = synth.init_positions(t, params, data, off, C, seed=N).astype(np.float32)
    prof = bsi.N.PROFILE_EXPONENTIAL if profile == "exp" else bsi.N.PROFILE_SPERGEL

    def run(n):
        rep = lambda x: np.concatenate([x] * (n // 2)).astype(np.float32)
        b = bsi.Batch(n=np.full(n, N), psf_fwhm=torch.tensor(rep(t.psf_fwhm)).cuda(),
                      sigma=torch.tensor(rep(t.sigma)).cuda(), pixel_scale=gen.PIXEL_SCALE, profile=prof)
        how = dict(sampler=bsi.N.SAMPLER_NUTS) if L == "nuts" else dict(n_leapfrog=L, jitter=jitter)
        cfg = bsi.HmcConfig(n_chains=C, n_warmup=warmup, n_samples=draws, adapt=True, step_size=0.003, seed=5,
                            **how)
        ref = torch.tensor(rep(np.stack([t.dx, t.dy], 1))).cuda()
        out = bsi.hmc_sample(b, torch.tensor(rep(data)).cuda(), ref, torch.tensor(rep(init)).cuda(), cfg)
        return [None if o is None else o[:2].cpu().numpy() for o in out]

    few, many = run(2), run(MANY)
    assert few[0].shape == (2, C, draws, 6) and np.all(np.isfinite(few[0]))
    assert np.any(few[0][:, :, 0] != few[0][:, :, -1])
    for a, b in zip(few, many):
        assert (a is None and b is None) or np.array_equal(a, b)
