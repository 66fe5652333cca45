"""Screens synthesised several to a launch: paths whose screens need more than
one such launch (24 screens at most, and 32 MiB of scratch), with a last launch
only partly full, forward and adjoint (which enters each batch from its last
screen) against the FP64 oracle, and the fused AR step against the two-call
one.  The bounds are the oracle tests' 1e-4 and, between two FP32 forms of the
same step, 1e-5."""
import numpy as np
import pytest
import torch

from oracle import propagate as opr
from paper_2604_07248_amd import workloads

from gpu_helpers import TOL, oracle_screens, rel_l2, say

pytestmark = pytest.mark.gpu


def _path(n, r, m, sh):
    dx = 4e-3 if n < 128 else 2e-3
    length = min(0.5 * n * dx * dx / 1e-6 * m, 3000.0)
    return workloads.uniform_path(n, n * dx, 1e-6, length, m, 1e-15, 0.005, 20.0, sh, realizations=r)


# 64: 24 + 2 screens; 1024, one pair: 4 + 1 screens; 512, two pairs: 8 + 3
@pytest.mark.parametrize("n,r,m,sh", [(64, 3, 26, 3), (512, 3, 11, 0), (1024, 2, 5, 0)])
def test_batches_match_oracle(gpu_lib, n, r, m, sh):
    from paper_2604_07248_amd import api
    path = _path(n, r, m, sh)
    plan = api.Plan(path)
    u0 = workloads.gaussian_source(n, path.dx, 0.1 * n * path.dx).astype(np.complex64)
    g = workloads.seeded_field((r, n, n), 3)
    dev = torch.from_numpy(u0).cuda()
    out, ck = plan.propagate(dev, seed=5, t=2, checkpoints=True)
    plain = plan.propagate(dev, seed=5, t=2)
    g_in, g_phi = plan.propagate_backward(torch.from_numpy(g).cuda(), ck, seed=5, t=2)
    phi = oracle_screens(path, 5, list(range(r)), t=2)
    ref, ref_ck = opr.propagate(u0.astype(np.complex128), path, phi)
    ref_in, ref_phi = opr.propagate_adjoint(g.astype(np.complex128), path, phi, ref_ck)
    errs = [rel_l2(a.cpu().numpy(), b) for a, b in ((out, ref), (plain, ref), (ck, ref_ck), (g_in, ref_in),
                                                    (g_phi, ref_phi), (plan.screens(5, t=2), phi))]
    say(f"[synth batch] n={n} R={r} M={m}: " + " ".join(f"{e:.1e}" for e in errs))
    assert max(errs) < TOL
    plan.close()


@pytest.mark.parametrize("n,r,m,sh", [(64, 3, 26, 3), (1024, 1, 6, 0)])
def test_fused_ar_step_equals_two_calls(gpu_lib, n, r, m, sh):
    from paper_2604_07248_amd import api
    path = _path(n, r, m, sh)
    plan = api.Plan(path)
    u0 = torch.from_numpy(workloads.gaussian_source(n, path.dx, 0.1 * n * path.dx).astype(np.complex64)).cuda()
    a, b = plan.init_spectra(seed=9), plan.init_spectra(seed=9)
    fused = plan.evolve_propagate(a, 9, 1, 0.9, 0.5, -0.25, u_in=u0)
    plan.evolve(b, 9, 1, 0.9, 0.5, -0.25)
    two = plan.propagate(u0, spectra=b)
    assert rel_l2(a.cpu().numpy(), b.cpu().numpy()) < 1e-5
    assert rel_l2(fused.cpu().numpy(), two.cpu().numpy()) < 1e-5
    plan.close()
