"""Subharmonics along the screen rows: every number of levels on both sides of
N = 64, from where four lanes of a row share the levels out, on the row
schedules of small and of larger counts and for a single realization's real
screen.  Bound: the oracle tests' 1e-4; a level left out, doubled or taken from
another lane changes a screen by several per cent."""
import numpy as np
import pytest
import torch

from paper_2604_07248_amd import workloads

from gpu_helpers import TOL, oracle_propagate, oracle_screens, rel_l2, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("levels", [1, 2, 3])
@pytest.mark.parametrize("n,r", [(16, 3), (32, 1), (32, 2), (64, 1), (64, 3), (128, 2), (256, 1), (256, 40), (512, 1)])
def test_levels(gpu_lib, n, r, levels):
    from paper_2604_07248_amd import api
    dx = 4e-3 if n < 128 else 2e-3
    path = workloads.uniform_path(n, n * dx, 1e-6, min(1.6 * n * dx * dx / 1e-6, 2000.0), 2, 1e-15, 0.005, 20.0,
                                  levels, realizations=r)
    say(f"[subharmonics] n={n} R={r} levels={levels}")
    some = sorted({0, r // 2, r - 1})
    phi = oracle_screens(path, 8, some, t=2)
    u0 = workloads.gaussian_source(n, dx, 0.1 * n * dx).astype(np.complex64)
    ref = oracle_propagate(path, 8, u0, realizations=some, screens=phi, t=2)[0]
    plan = api.Plan(path)
    dev = torch.from_numpy(u0).cuda()
    plain = plan.propagate(dev, seed=8, t=2)
    kept, _ = plan.propagate(dev, seed=8, t=2, checkpoints=True)
    errs = [rel_l2(a.cpu().numpy()[some], b)
            for a, b in ((plan.screens(8, 2), phi), (plain, ref), (kept, ref))]
    say("[subharmonics] screens, fields, with checkpoints: " + " ".join(f"{e:.1e}" for e in errs))
    plan.close()
    assert max(errs) < TOL
