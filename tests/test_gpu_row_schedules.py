"""The row pass with one worker per transform (launches of at most 2^20 scratch
pixels) against the schedules of larger launches: realization r of a path
draws the same noise whatever the count, so the fields, checkpoints and
gradients of the first realizations must be the same bits on both sides of the
line.  Counts at the line and the next one above, an odd count among them, and
both against the FP64 oracle on one realization."""
import numpy as np
import pytest
import torch

from paper_2604_07248_amd import workloads

from gpu_helpers import TOL, oracle_propagate, rel_l2, say

pytestmark = pytest.mark.gpu


# (n, count at the line, count above it): ceil(count / 2) n^2 = 2^20 at the line
@pytest.mark.parametrize("n,low,high,sh", [(64, 511, 514, 3), (128, 127, 130, 0), (256, 32, 33, 3), (512, 7, 10, 0),
                                           (1024, 2, 3, 2)])
def test_same_bits_on_both_sides_of_the_line(gpu_lib, n, low, high, sh):
    from paper_2604_07248_amd import api
    api.tune_cache_clear()  # a tuned radix plan of one count's class would round differently from the other's
    m, dx = 2, 4e-3 if n < 128 else 2e-3
    base = workloads.uniform_path(n, n * dx, 1e-6, min(0.8 * n * dx * dx / 1e-6 * m, 2000.0), m, 1e-15, 0.005, 20.0, sh)
    src = torch.from_numpy(workloads.seeded_field((4, n, n), 1)).cuda()
    cot = torch.from_numpy(workloads.seeded_field((4, n, n), 2)).cuda()
    got = []
    for r in (low, high):
        plan = api.Plan(base.with_(realizations=r))
        own = src.repeat((r + 3) // 4, 1, 1)[:r].contiguous()
        g = cot.repeat((r + 3) // 4, 1, 1)[:r].contiguous()
        plain = plan.propagate(own, seed=8, t=1)
        shared = plan.propagate(src[0].contiguous(), seed=8, t=1)
        out, ck = plan.propagate(own, seed=8, t=1, checkpoints=True)
        g_in, g_phi = plan.propagate_backward(g, ck, seed=8, t=1)
        rev_in, rev_phi = plan.propagate_backward(g, None, seed=8, t=1, u_out=out)
        got.append([x[:low] for x in (plain, shared, out, ck, g_in, g_phi, rev_in, rev_phi)])
        plan.close()
    last = low - 1
    ref = oracle_propagate(base.with_(realizations=low), 8, own.cpu().numpy(), realizations=[last], t=1)[0]
    err = rel_l2(got[0][0][last].cpu().numpy(), ref[0])
    say(f"[row schedules] n={n} R={low}|{high}: oracle {err:.1e}")
    assert err < TOL
    names = ("plain", "shared", "out", "checkpoints", "g_in", "g_phi", "rev_in", "rev_phi")
    for name, a, b in zip(names, *got):
        assert torch.equal(a, b), name
