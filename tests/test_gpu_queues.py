"""The stamp sides of one sampling call, or of a request server, run side by side, on
the four hardware queues; those of a call also where the library's handle is the
first thing a process does on the device (a process of its own, which prints how
long the four sides took together and the longest of them alone)."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
import sys, time
import numpy as np, torch
from paper_2604_22048_amd import api
if sys.argv[1] == "tensors":
    torch.zeros(8, device="cuda").sum().item()
lib = api.Library(0)

def took(sides):
    G, C = len(sides), 2
    b = api.Batch(n=np.asarray(sides), psf_fwhm=torch.full((G,), 0.7, device="cuda"),
                  sigma=torch.ones(G, device="cuda"))
    p = torch.tensor([[800.0, 0.5, 0.1, 0.05, 0.1, -0.1]] * G, device="cuda")
    data = api.render_stamps(b, p, lib=lib)
    th = torch.stack([torch.log10(p[:, 0]), torch.log10(p[:, 1]), p[:, 2], p[:, 3], 0 * p[:, 0], 0 * p[:, 0]], 1)
    init = th[:, None].expand(G, C, 6).contiguous()
    cfg = api.HmcConfig(n_chains=C, n_leapfrog=20, n_warmup=0, n_samples=40, adapt=False, step_size=1e-3, seed=3,
                        metric=1, iters_per_launch=1000)
    best = 1e9
    for _ in range(4):
        torch.cuda.synchronize()
        t = time.perf_counter()
        api.hmc_sample(b, data, p[:, 4:6].contiguous(), init, cfg, lib=lib)
        torch.cuda.synchronize()
        best = min(best, time.perf_counter() - t)
    return best

sides = [104, 106, 108, 110]
print("together", took(sides), "longest", max(took([s]) for s in sides), flush=True)
"""


@pytest.mark.parametrize("first", ["handle", "tensors"])
def test_four_sides_run_side_by_side(device, first):
    out = subprocess.run([sys.executable, "-c", PROGRAM, first], cwd=ROOT, capture_output=True, text=True, timeout=100)
    assert out.returncode == 0, out.stderr[-2000:]
    w = out.stdout.split()
    together, longest = float(w[w.index("together") + 1]), float(w[w.index("longest") + 1])
    print(f"{first} first: together {together * 1e3:.2f} ms, longest alone {longest * 1e3:.2f} ms", flush=True)
    assert together < 1.5 * longest           # two on one queue: twice the longest


@pytest.mark.parametrize("sides,waves", [((104, 106, 108, 110), 1), ((53, 73, 101), 4)])
def test_sides_of_a_server_run_side_by_side(device, sides, waves):
    """One request of each side: an advance of all of them takes about as long as
    one of the longest alone (one after another: the sum)."""
    import time

    import torch

    from paper_2604_22048_amd import api

    def took(ns):
        cfg = api.HmcConfig(n_chains=1, n_leapfrog=20, n_warmup=0, n_samples=400, adapt=False, step_size=1e-3, seed=3,
                            metric=1, waves_per_chain=waves)
        srv = api.Slots(list(ns), cfg, hbm_budget=1 << 30, max_slots=8)
        p = torch.tensor([[800.0, 0.5, 0.1, 0.05, 0.1, -0.1]], device="cuda")
        for i, n in enumerate(ns):
            b = api.Batch(n=[n], psf_fwhm=torch.full((1,), 0.7, device="cuda"), sigma=torch.ones(1, device="cuda"))
            assert srv.admit(i, api.render_stamps(b, p), 0.7, 1.0, (0.1, -0.1), [2.9, -0.3, 0.1, 0.05, 0.0, 0.0])
        best = 1e9
        for _ in range(5):
            t = time.perf_counter()
            srv.advance(40)
            srv.poll()
            best = min(best, time.perf_counter() - t)
        srv.close()
        return best

    together, alone = took(sides), [took([n]) for n in sides]
    print(f"{sides}, {waves} waves a chain: together {together * 1e3:.2f} ms, alone {[round(a * 1e3, 2) for a in alone]}",
          flush=True)
    assert together < 0.5 * (max(alone) + sum(alone))
