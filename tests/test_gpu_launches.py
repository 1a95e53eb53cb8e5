"""A sampling call's iterations in several launches and in one: the same draws
and chain statistics, to the last bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from workloads import gen              # noqa: E402
from tests import synth                # noqa: E402


@pytest.fixture(scope="module")
def bsi(device):
    from paper_2604_22048_amd import api
    return api


# (sides, chains, slot plan): teams (a few galaxies of the specialised sides),
# one wave per chain group (other sides, other plans, more than four chains)
BATCHES = [([53] * 3, 4, 0), ([101, 73, 25], 1, 0), ([41, 53], 2, 0), ([32, 48], 2, 0), ([53, 25], 4, 4), ([53], 8, 0)]


@pytest.mark.parametrize("sides,C,plan", BATCHES)
@pytest.mark.parametrize("how", ["hmc", "nuts"])
def test_one_launch_draws_what_several_do(bsi, sides, C, plan, how):
    import torch
    print(f"launches {how} {sides} C={C} plan {plan}", flush=True)
    t, params, data, off = synth.make_population("uneven", n_gal=len(sides), seed=sides[0] + C, sizes=sides)
    init = synth.init_positions(t, params, data, off, C, seed=3).astype(np.float32)
    lib = bsi.Library(0)
    for n in set(sides) if plan else ():
        bsi.set_plan(n, plan, lib=lib)
    b = bsi.Batch(n=np.asarray(t.n_pix), psf_fwhm=torch.tensor(t.psf_fwhm.astype(np.float32)).cuda(),
                  sigma=torch.tensor(t.sigma.astype(np.float32)).cuda(), pixel_scale=gen.PIXEL_SCALE)
    ref = torch.tensor(np.stack([t.dx, t.dy], 1).astype(np.float32)).cuda()
    # 70 trajectories of 20 steps, 40 transitions: more than 512 evaluations' worth
    W, S = (30, 40) if how == "hmc" else (17, 23)
    cfg = dict(n_chains=C, n_leapfrog=20, n_warmup=W, n_samples=S, adapt=True, step_size=0.003, seed=7,
               metric=bsi.N.METRIC_FISHER,
               sampler=bsi.N.SAMPLER_NUTS if how == "nuts" else bsi.N.SAMPLER_HMC)

    def run(ipl):
        trace = torch.full((len(sides), C, W + S, 4), float("nan"), device="cuda")
        out = bsi.hmc_sample(b, torch.tensor(data).cuda(), ref, torch.tensor(init).cuda(),
                             bsi.HmcConfig(iters_per_launch=ipl, **cfg), trace=trace, lib=lib)
        return [x.cpu().numpy() for x in (*out, trace)]

    several = run(1)
    # (dH of a trajectory that left the support is not finite; its acceptance statistic is 0)
    written = bool(np.isfinite(several[0]).all() and np.isfinite(several[3][..., 2]).all())
    assert written
    assert np.any(several[0][:, :, 0] != several[0][:, :, -1])
    for ipl in (W + S, 2**31 - 1):
        for x, y in zip(several, run(ipl)):
            same = np.array_equal(x, y, equal_nan=True)
            assert same, ipl
    lib.close()
