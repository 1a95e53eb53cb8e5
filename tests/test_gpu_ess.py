"""bsi_ess at the edges of its layout: runs of 5, 9 and 17 draws per lane, 64 runs
per wave round, 16 lags per pass over the chains, parameters per workgroup, and
the chains shared by several waves up to 3,072 series."""
import numpy as np
import pytest

from oracle import diagnostics

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bsi(device):
    from paper_2604_22048_amd import api
    return api


# (galaxies, chains, draws, parameters, memory of the chains in draws)
SHAPES = [(3, 1, 4, 1, 0), (2, 16, 15, 6, 0), (2, 2, 16, 5, 1), (3, 4, 17, 9, 2), (1, 4, 1024, 6, 3),
          (2, 2, 1041, 7, 40), (1, 3, 2500, 6, 200), (1, 1, 18944, 2, 30),
          (1, 11, 321, 3, 0), (3100, 2, 33, 1, 1), (1600, 1, 320, 2, 0), (800, 3, 577, 4, 2), (400, 2, 90, 8, 30),
          (400, 2, 600, 9, 0), (700, 2, 1089, 5, 4),
          (100, 1, 200, 6, 3), (30, 1, 2000, 7, 20)]


@pytest.mark.parametrize("G,C,S,P,memory", SHAPES)
def test_ess_layout_edges(bsi, G, C, S, P, memory):
    """Every float64 sum here is good to about 1e-13 of its value, so what is left
    of the difference is the float32 rounding of the result (2^-24; twice that
    allowed)."""
    import torch
    rng = np.random.default_rng(G + 100 * C + 1000 * S)
    x = rng.normal(size=(G, C, S + 4 * memory, P))
    if memory:
        r = np.exp(-1.0 / memory)
        for t in range(1, x.shape[2]):
            x[:, :, t] += r * x[:, :, t - 1]
    x = (x[:, :, 4 * memory:] + rng.normal(size=(G, C, 1, P)) * 0.05 + 3.0).astype(np.float32)
    e, r, rs = [a.cpu().numpy().astype(np.float64) for a in bsi.ess(torch.tensor(x).cuda(), split=True)]
    e2 = bsi.ess(torch.tensor(x).cuda())[0].cpu().numpy()
    assert np.array_equal(e2, e.astype(np.float32))
    tol = 2.0 ** -23
    for g in sorted({0, G // 2, G - 1}):
        for p in range(P):
            y = x[g, :, :, p].astype(np.float64)
            assert abs(e[g, p] / diagnostics.ess(y) - 1) < tol
            if C > 1:
                assert abs(r[g, p] / diagnostics.rhat(y) - 1) < tol
            assert abs(rs[g, p] / diagnostics.split_rhat(y) - 1) < tol


def test_ess_constant_chains(bsi):
    """No variance at all: the number of draws; no variance within the chains
    only: every lag is taken, to the last pair."""
    import torch
    x = torch.zeros(2, 2, 100, 2)
    x[1, 1] = 0.5
    e, _ = bsi.ess(x.cuda())
    assert torch.all(e[0] == 200)
    # rho = 1 at every lag: tau = -1 + 2 (2 S / 2) = 199
    assert torch.allclose(e[1].cpu(), torch.full((2,), 200 / 199.0), rtol=2.0 ** -23)


@pytest.mark.parametrize("G,C,S,P", [(2, 1, 5, 6), (3, 2, 7, 1), (2, 3, 333, 9), (700, 4, 601, 6)])
@pytest.mark.parametrize("value", [float("nan"), float("inf"), -float("inf"), 1e30])
def test_split_rhat_leaves_the_middle_draw_out(bsi, G, C, S, P, value):
    """An odd chain's middle draw is in neither half, whatever it holds."""
    import torch
    x = np.random.default_rng(S).normal(size=(G, C, S, P)).astype(np.float32)
    y = x.copy()
    y[0, 0, S // 2, 0] = y[-1, -1, S // 2, -1] = value
    rs = bsi.ess(torch.tensor(x).cuda(), split=True)[2].cpu().numpy()
    out = [a.cpu().numpy() for a in bsi.ess(torch.tensor(y).cuda(), split=True)]
    assert np.array_equal(out[2], rs)
    assert np.isfinite(out[0][-1, -1]) == (abs(value) < 1e31) or out[0][-1, -1] == C * S


# slowly mixing chains, whose scan goes on for many blocks of 16 lags: one to eight
# waves a series, blocks side by side, galaxies that do not fill the XCDs' turns
@pytest.mark.parametrize("G,C,S,P,memory", [(9, 2, 100, 5, 50), (100, 2, 100, 5, 80), (17, 4, 300, 20, 60),
                                            (1, 1, 2000, 1, 400), (41, 8, 500, 3, 100), (1030, 4, 60, 2, 10),
                                            (601, 3, 1000, 6, 30), (1, 16, 1184, 6, 50), (2051, 1, 257, 2, 40)])
def test_ess_of_slowly_mixing_chains(bsi, G, C, S, P, memory):
    test_ess_layout_edges(bsi, G, C, S, P, memory)


@pytest.mark.parametrize("G,C,S,P", [(3, 2, 40, 3), (700, 4, 1000, 6)])
def test_ess_outputs_alone(bsi, G, C, S, P):
    """Each output is the same whichever others are asked for."""
    import torch
    x = torch.randn(G, C, S, P, device="cuda", generator=torch.Generator("cuda").manual_seed(1))
    want = bsi.ess(x, split=True)
    lib = bsi.get(0)
    for i in range(3):
        out = [None, None, None]
        out[i] = torch.full((G, P), -7.0, device="cuda")
        lib.check(lib.lib.bsi_ess(lib.h, G, C, S, P, x.data_ptr(), *[None if o is None else o.data_ptr() for o in out],
                                  None), "bsi_ess")
        torch.cuda.synchronize()
        same = torch.equal(out[i], want[i])
        assert same, i
