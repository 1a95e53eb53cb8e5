"""Pixels of api.render_stamps that no galaxy's stamp covers are zero: gaps
between stamps, and stamps past the last galaxy's exposures."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,n_exp,off", [([16] * 3, 2, None), ([16, 16, 12, 12, 9], 2, None), ([8] * 5, 3, None),
                                         ([16, 16], 1, [0, 300]), ([16, 16], 1, [44, 300]), ([12, 12], 2, [200, 0])])
def test_uncovered_pixels_are_zero(device, n, n_exp, off):
    import torch
    from paper_2604_22048_amd import api
    n = np.asarray(n)
    b = api.Batch(n=n, psf_fwhm=torch.full((len(n),), 0.7, device="cuda"), sigma=torch.ones(len(n), device="cuda"),
                  off=None if off is None else np.asarray(off), n_exp=n_exp)
    p = torch.tensor([[500.0, 0.5, 0.1, -0.05, 0.2, -0.3]] * b.n_gal, device="cuda")
    covered = np.zeros(b.n_pixels, bool)
    for i in range(b.n_gal * n_exp):
        covered[b.off[i]:b.off[i] + n[i] ** 2] = True
    assert not covered.all()
    used = torch.full((b.n_pixels,), float("nan"), device="cuda")    # what a recycled block holds
    del used
    out = api.render_stamps(b, p).cpu().numpy()
    assert np.all(out[~covered] == 0) and np.all(np.isfinite(out[covered])) and np.any(out[covered] != 0)
