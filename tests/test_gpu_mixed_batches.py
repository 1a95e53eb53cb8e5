"""Batches of several stamp sides, whose sizes run one after another or, where
that is longer than the forked streams take, side by side: each galaxy's log
likelihood, gradient and render are those of a batch of its own, to the bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from workloads import gen              # noqa: E402


@pytest.fixture(scope="module")
def bsi(device):
    from paper_2604_22048_amd import api
    return api


def _batch(bsi, sides, E, seed):
    import torch
    rng = np.random.default_rng(seed)
    n = np.repeat(sides, E)
    b = bsi.Batch(n=n, psf_fwhm=torch.tensor(rng.uniform(0.6, 0.9, len(n)).astype(np.float32)).cuda(),
                  sigma=torch.tensor(rng.uniform(0.5, 1.5, len(n)).astype(np.float32)).cuda(),
                  pixel_scale=gen.PIXEL_SCALE, n_exp=E)
    G = len(sides)
    p = np.stack([rng.uniform(200, 2000, G), rng.uniform(0.3, 0.9, G), rng.uniform(-0.3, 0.3, G),
                  rng.uniform(-0.3, 0.3, G), rng.uniform(-0.5, 0.5, G), rng.uniform(-0.5, 0.5, G)], 1)
    return b, torch.tensor(p.astype(np.float32)).cuda()


# (galaxies, sides, exposures, method): in sequence, then forked
CASES = [(3, [25, 41, 53], 1, "kspace"), (40, [16, 33, 64], 1, "kspace"), (60, [25, 41, 53, 73, 101], 3, "kspace"),
         (400, [41, 64, 101, 127], 1, "kspace"), (4, [25, 53], 1, "pixel"), (300, [30, 53, 90], 1, "pixel")]


@pytest.mark.parametrize("G,sides,E,method", CASES)
def test_mixed_batch_is_its_galaxies(bsi, G, sides, E, method):
    import torch
    how = bsi.N.LIK_PIXEL if method == "pixel" else bsi.N.LIK_KSPACE
    rng = np.random.default_rng(G)
    s = rng.choice(sides, G)
    s[:len(sides)] = sides
    b, p = _batch(bsi, s, E, G + 1)
    m = bsi.render_stamps(b, p)
    data = m + torch.randn(m.shape, device="cuda", generator=torch.Generator("cuda").manual_seed(2))
    ll, gr, st = bsi.loglik_grad(b, data, p, method=how)
    for i in list(range(len(sides))) + [G - 1]:
        o, e = int(b.off[i * E]), int(b.off[i * E + E - 1]) + int(s[i]) ** 2
        one = bsi.Batch(n=b.n[i * E:i * E + E], psf_fwhm=b.psf_fwhm[i * E:i * E + E], sigma=b.sigma[i * E:i * E + E],
                        pixel_scale=gen.PIXEL_SCALE, n_exp=E)
        m1 = bsi.render_stamps(one, p[i:i + 1])
        ll1, gr1, st1 = bsi.loglik_grad(one, data[o:e].contiguous(), p[i:i + 1], method=how)
        same = (torch.equal(m1, m[o:e]) and torch.equal(ll1, ll[i:i + 1]) and torch.equal(gr1, gr[i:i + 1])
                and torch.equal(st1, st[i:i + 1]))
        assert same, i
