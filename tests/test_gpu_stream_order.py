"""Calls of one handle on two streams run in the order they are made ("Workspace,
streams and graph capture" of include/bsi.h), also those that need none of its
workspace: packed batches of one stamp side."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from workloads import gen              # noqa: E402
from tests import synth                # noqa: E402


@pytest.fixture(scope="module")
def bsi(device):
    from paper_2604_22048_amd import api
    return api


def _setup(bsi, N, G, C):
    import torch
    t, params, data, off = synth.make_population("uneven", n_gal=G, seed=N, sizes=[N] * G)
    init = synth.init_positions(t, params, data, off, C, seed=5).astype(np.float32)
    b = bsi.Batch(n=np.asarray(t.n_pix), psf_fwhm=torch.tensor(t.psf_fwhm.astype(np.float32)).cuda(),
                  sigma=torch.tensor(t.sigma.astype(np.float32)).cuda(), pixel_scale=gen.PIXEL_SCALE)
    ref = torch.tensor(np.stack([t.dx, t.dy], 1).astype(np.float32)).cuda()
    cfg = bsi.HmcConfig(n_chains=C, n_leapfrog=10, n_warmup=5, n_samples=10, adapt=True, step_size=0.01, seed=3,
                        metric=bsi.N.METRIC_FISHER)
    return b, torch.tensor(params.astype(np.float32)).cuda(), torch.tensor(data).cuda(), ref, \
        torch.tensor(init).cuda(), cfg


def _busy(torch, x):
    """Some tens of milliseconds of work on the current stream."""
    for _ in range(20):
        x = x @ x
    return x


@pytest.mark.parametrize("N", [25, 53])
def test_packed_render_on_one_stream_sampled_on_another(bsi, N):
    import torch
    lib = bsi.Library(0)
    b, p, _, ref, init, cfg = _setup(bsi, N, 6, 2)
    want = bsi.hmc_sample(b, bsi.render_stamps(b, p, lib=lib), ref, init, cfg, lib=lib)[0]
    torch.cuda.synchronize()
    a = torch.zeros(8192, 8192, device="cuda")
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    for _ in range(2):
        with torch.cuda.stream(s1):
            _busy(torch, a)
            m = bsi.render_stamps(b, p, lib=lib)
        with torch.cuda.stream(s2):
            got = bsi.hmc_sample(b, m, ref, init, cfg, lib=lib)[0]
        torch.cuda.synchronize()
        same = torch.equal(got, want)
        assert same
        m.zero_()                 # (the block's next tenant, if it is this one, starts from zeros)
        del m
        torch.cuda.synchronize()
    lib.close()


@pytest.mark.parametrize("N", [25, 53])
def test_packed_loglik_after_a_call_on_another_stream(bsi, N):
    """render (busy stream) -> loglik of its stamps -> sampler on the first
    stream's data: each call waits for the one before it."""
    import torch
    lib = bsi.Library(0)
    b, p, data, ref, init, cfg = _setup(bsi, N, 6, 2)
    m0 = bsi.render_stamps(b, p, lib=lib)
    want = bsi.loglik_grad(b, m0, p, lib=lib)[:2]
    torch.cuda.synchronize()
    a = torch.zeros(8192, 8192, device="cuda")
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    for _ in range(2):
        with torch.cuda.stream(s1):
            _busy(torch, a)
            m = bsi.render_stamps(b, p, lib=lib)
        with torch.cuda.stream(s2):
            got = bsi.loglik_grad(b, m, p, lib=lib)[:2]
            _busy(torch, a)
            last = bsi.loglik_grad(b, data, p, lib=lib)[0]
        with torch.cuda.stream(s1):
            # a call behind the busy stream's: reads what it wrote
            copy = torch.empty_like(p)
            copy.copy_(p)
            bsi.render_stamps(b, copy, lib=lib)
            seen = last.clone()
        torch.cuda.synchronize()
        same = all(torch.equal(x, y) for x, y in zip(got, want)) and torch.equal(seen, last)
        assert same
        m.zero_()
        last.zero_()
        del m, last
        torch.cuda.synchronize()
    lib.close()
