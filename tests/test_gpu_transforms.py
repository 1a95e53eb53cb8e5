"""The transform kernels where their layouts change: sides around multiples of 16
(and of 8 in the last block of frequencies), one, two and four units per wave,
packed batches and batches with gaps, transform and contraction in one kernel
or in two."""
import numpy as np
import pytest

from oracle import render

pytestmark = pytest.mark.gpu

SIDES = [8, 9, 12, 15, 16, 17, 31, 32, 33, 46, 47, 48, 49, 63, 64, 65, 80, 96, 112, 113, 127, 128]


@pytest.fixture(scope="module")
def bsi(device):
    from paper_2604_22048_amd import api
    return api


def _batch(bsi, n, gap=0, **kw):
    import torch
    n = np.asarray(n, np.int32)
    size = n.astype(np.int64) ** 2
    off = np.concatenate([[0], np.cumsum(size + gap)[:-1]]).astype(np.int64) + gap
    G = len(n)
    return bsi.Batch(n=n, off=off, psf_fwhm=torch.linspace(0.6, 0.9, G).cuda(), sigma=torch.linspace(0.8, 1.2, G).cuda(),
                     **kw)


def _params(G, seed):
    rng = np.random.default_rng(seed)
    p = np.stack([rng.uniform(200, 2000, G), rng.uniform(0.3, 0.9, G), *rng.uniform(-0.4, 0.4, (2, G)),
                  *rng.uniform(-1, 1, (2, G))], 1)
    return p.astype(np.float32)


@pytest.mark.parametrize("N", SIDES)
def test_render_and_pixel_likelihood(bsi, N):
    """Stamps within 1e-5 of the peak (the renderer's bar) and the float64 pixel
    likelihood: its model carries the float64 rounding of sums of at most 2 x 65
    terms of the peak's size, below 1e-13 of the peak, against residuals of
    about one; 1e-10 of log L leaves room for the float32 PSF and scale
    constants, which enter the model at 6e-8 of the derivative of log L."""
    import torch
    p = _params(3, N)
    b = _batch(bsi, [N] * 3)
    out = bsi.render_stamps(b, torch.tensor(p).cuda()).cpu().numpy()
    fw, sg = b.psf_fwhm.cpu().numpy().astype(np.float64), b.sigma.cpu().numpy().astype(np.float64)
    rng = np.random.default_rng(N)
    data = np.empty(out.shape, np.float32)
    models = []
    for i in range(3):
        at = slice(int(b.off[i]), int(b.off[i]) + N * N)
        m = render.render_one(p[i].astype(np.float64), N, 0.2, fw[i])
        models.append(m)
        assert np.max(np.abs(out[at] - m.ravel())) <= 1e-5 * np.max(np.abs(m))
        data[at] = m.ravel() + sg[i] * rng.normal(size=N * N)
    ll, g, _ = bsi.loglik_grad(b, torch.tensor(data).cuda(), torch.tensor(p).cuda(), method=bsi.N.LIK_PIXEL)
    for i in range(3):
        d = data[int(b.off[i]):int(b.off[i]) + N * N].astype(np.float64).reshape(N, N)
        ref, gr = render.loglik_grad(d, p[i].astype(np.float64), N, 0.2, fw[i], sg[i])
        dm = 1e-7 * np.sum(np.abs(gr) * np.abs(p[i])) + 1e-6 * abs(gr[1] * p[i][1])
        assert abs(ll[i].item() - ref) <= 1e-10 * abs(ref) + dm


@pytest.mark.parametrize("N", SIDES)
def test_packed_and_gapped_batches_agree(bsi, N):
    """The index-list-free path of packed batches against the general one: same
    kernels, same bits; gaps come back zero."""
    import torch
    p = torch.tensor(_params(5, N + 1)).cuda()
    a, c = _batch(bsi, [N] * 5), _batch(bsi, [N] * 5, gap=3)
    xa, xc = bsi.render_stamps(a, p), bsi.render_stamps(c, p)
    take = lambda x, b: torch.stack([x[int(o):int(o) + N * N] for o in b.off])      # noqa: E731
    assert torch.equal(take(xa, a), take(xc, c))
    assert torch.count_nonzero(xc[:3]) == 0 and torch.count_nonzero(xc[int(c.off[1]) - 3:int(c.off[1])]) == 0
    da, dc = xa + torch.randn_like(xa), torch.full_like(xc, float("nan"))
    for i in range(5):
        dc[int(c.off[i]):int(c.off[i]) + N * N] = take(da, a)[i]
    for method in (bsi.N.LIK_KSPACE, bsi.N.LIK_PIXEL):
        for u, v in zip(bsi.loglik_grad(a, da, p, method=method), bsi.loglik_grad(c, dc, p, method=method)):
            assert torch.equal(u, v)


@pytest.mark.parametrize("N,E", [(66, 1), (73, 1), (73, 2), (101, 3), (128, 1)])
def test_one_kernel_and_two_agree(bsi, N, E):
    """Beyond 1,024 stamps of a larger side the spectra go through memory: the
    first galaxies of a large batch against the same galaxies alone."""
    import torch
    G = 1100 // E
    p = torch.tensor(_params(G, N)).cuda()
    big, few = _batch(bsi, [N] * (G * E), n_exp=E), _batch(bsi, [N] * (G * E), n_exp=E)
    few.n, few.off = few.n[:4 * E], few.off[:4 * E]
    data = torch.randn(G * E * N * N, device="cuda", generator=torch.Generator("cuda").manual_seed(N))
    for u, v in zip(bsi.loglik_grad(big, data, p), bsi.loglik_grad(few, data, p[:4].contiguous())):
        assert torch.equal(u[:4], v)
