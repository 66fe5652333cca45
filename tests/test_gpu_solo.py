"""A single realization, whose real screen is synthesised on its own (Hermitian
half of the spectrum, two rows to a complex one): every grid size it is built
for and the one below, forward, checkpointed forward, both adjoints, with and
without subharmonics, and against a plan whose screens stay with the
checkpoints (full complex planes).  Bounds: the oracle tests' 1e-4; between the
two FP32 forms of the screens, which differ by rounding only, 1e-5."""
import numpy as np
import pytest
import torch

from oracle import propagate as opr
from paper_2604_07248_amd import binding as B
from paper_2604_07248_amd import workloads

from gpu_helpers import TOL, oracle_screens, rel_l2, say

pytestmark = pytest.mark.gpu


def _path(n, m, sh):
    dx = 4e-3 if n < 128 else 2e-3
    length = min(0.8 * n * dx * dx / 1e-6 * m, 2000.0)
    return workloads.uniform_path(n, n * dx, 1e-6, length, m, 1e-15, 0.005, 20.0, sh, realizations=1)


@pytest.mark.parametrize("n,m,sh", [(32, 3, 3), (64, 27, 3), (64, 2, 0), (128, 3, 0), (256, 3, 3), (512, 2, 0),
                                    (1024, 2, 1), (2048, 3, 2)])
def test_single_realization(gpu_lib, n, m, sh):
    from paper_2604_07248_amd import api
    path = _path(n, m, sh)
    u0 = workloads.gaussian_source(n, path.dx, 0.1 * n * path.dx).astype(np.complex64)
    g = workloads.seeded_field((1, n, n), 4)
    phi = oracle_screens(path, 6, [0], t=3)
    ref, ref_ck = opr.propagate(u0.astype(np.complex128), path, phi)
    ref_in, ref_phi = opr.propagate_adjoint(g.astype(np.complex128), path, phi, ref_ck)
    dev, gdev = torch.from_numpy(u0).cuda(), torch.from_numpy(g).cuda()
    plans = [api.Plan(path), api.Plan(path, flags=B.SCREEN_CHECKPOINTS)]
    outs = []
    for plan in plans:
        plain = plan.propagate(dev, seed=6, t=3)
        own = plan.propagate(dev[None].contiguous(), seed=6, t=3)
        out, ck = plan.propagate(dev, seed=6, t=3, checkpoints=True)
        g_in, g_phi = plan.propagate_backward(gdev, ck, seed=6, t=3)
        shared, _ = plan.propagate_backward(gdev, ck, seed=6, t=3, shared_source=True)
        rev_in, rev_phi = plan.propagate_backward(gdev, None, seed=6, t=3, u_out=out)
        got = [plain, own, out, plan.checkpoint_fields(ck), g_in, g_phi, shared[None], rev_in, rev_phi]
        want = [ref, ref, ref, ref_ck, ref_in, ref_phi, ref_in, ref_in, ref_phi]
        errs = [rel_l2(a.cpu().numpy(), b) for a, b in zip(got, want)]
        say(f"[solo] n={n} M={m} sh={sh}: " + " ".join(f"{e:.1e}" for e in errs))
        assert max(errs) < TOL
        outs.append([a.cpu().numpy() for a in got])
    assert max(rel_l2(a, b) for a, b in zip(*outs)) < 1e-5
    static = torch.empty((1, n, n), dtype=torch.complex64, device="cuda")
    if B.workspace_size(plans[0].handle, B.OP_PROPAGATE) <= 64 << 20:
        B.check(B.lib().turpy_propagate_static(plans[0].handle, 6, 3, api._ptr(dev), 0, 0, None, api._ptr(static), None,
                                               api._stream()))
        assert np.array_equal(static.cpu().numpy(), outs[0][0])
    for plan in plans:
        plan.close()
