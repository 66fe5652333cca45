"""The tuner against the launches that calls make: the synthesis is timed with
as many screens as a call's launch covers, and what it chose goes only to plans
whose launches are alike.  The row passes' occupancy hint is timed on the
schedules that take one."""
import ctypes

import pytest
import torch

from paper_2604_07248_amd import binding as B
from paper_2604_07248_amd import workloads

from gpu_helpers import rel_l2, say

pytestmark = pytest.mark.gpu


@pytest.fixture
def api(gpu_lib):
    from paper_2604_07248_amd import api as _api
    _api.tune_cache_clear()
    yield _api
    _api.tune_cache_clear()


def _path(n, r, m, sh=0):
    dx = 4e-3 if n < 128 else 2e-3
    return workloads.uniform_path(n, n * dx, 1e-6, min(0.5 * n * dx * dx / 1e-6 * m, 2000.0), m, 1e-15, 0.005, 20.0, sh,
                                  realizations=r)


def _entry(api, kernel):
    return [e for e in api.tune_cache() if e["kernel"] == kernel]


# (n, R, M): class of the synthesis, of the AR step.  512, 4 pairs and two
# screens fill the chip; one pair with one screen, or with six of a small grid,
# does not; a single realization has its own kernel, but not for stored spectra
@pytest.mark.parametrize("n,r,m,synth,ar", [(512, 8, 2, 3, 3), (256, 2, 1, 33, 33), (256, 2, 6, 35, 35),
                                            (256, 1, 6, 51, 35), (1024, 1, 1, 49, 33), (1024, 2, 5, 1, 1)])
def test_classes_and_results(api, n, r, m, synth, ar):
    path = _path(n, r, m, 3)
    plan = api.Plan(path)
    u0 = torch.from_numpy(workloads.seeded_field((n, n), 31)).cuda()
    state = plan.init_spectra(4)
    ref = plan.propagate(u0, seed=4)
    ref_ar = plan.evolve_propagate(state, 4, 1, 0.9, 0.5, -0.25, u_in=u0)
    plan.tune()
    assert [e["batch_class"] for e in _entry(api, "synth")] == [synth]
    assert [e["batch_class"] for e in _entry(api, "synth_ar")] == [ar]
    say(f"[tune] n={n} R={r} M={m}: {_entry(api, 'synth')} {_entry(api, 'synth_ar')}")
    assert rel_l2(plan.propagate(u0, seed=4).cpu().numpy(), ref.cpu().numpy()) < 1e-5
    state = plan.init_spectra(4)
    got = plan.evolve_propagate(state, 4, 1, 0.9, 0.5, -0.25, u_in=u0)
    assert rel_l2(got.cpu().numpy(), ref_ar.cpu().numpy()) < 1e-5
    plan.close()


def test_choices_go_to_plans_with_like_launches(api):
    """A single realization, a pair with one screen and a pair with many screens
    run different launches: what is put for one leaves the others alone."""
    arch = torch.cuda.get_device_properties(0).gcnArchName.split(":")[0]
    paths = {"solo": _path(256, 1, 6), "one": _path(256, 2, 1), "many": _path(256, 2, 24)}
    before = {k: api.Plan(p).config for k, p in paths.items()}
    classes = {}
    for k, p in paths.items():
        api.tune_cache_clear()
        api.Plan(p).tune()
        classes[k] = _entry(api, "synth")[0]["batch_class"], _entry(api, "synth_ar")[0]["batch_class"]
    assert len({c[0] for c in classes.values()}) == 3
    for k in paths:
        api.tune_cache_clear()
        other = 4 if before[k]["synth_width"] != 4 else 16
        B.tune_cache_put([{"arch": arch, "kernel": "synth", "n": 256, "batch_class": classes[k][0], "width": other}])
        for j, p in paths.items():
            assert api.Plan(p).config["synth_width"] == (other if j == k else before[j]["synth_width"]), (k, j)


def test_tuning_stays_in_its_workspace(api):
    """Small plans, whose AR launches cover many screens at once."""
    for n, r, m in ((64, 2, 24), (256, 1, 24), (16, 3, 5)):
        plan = api.Plan(_path(n, r, m))
        size, guard = B.workspace_size(plan.handle, B.OP_TUNE), 1 << 20
        ws = torch.full((size + guard,), 0xA5, dtype=torch.uint8, device="cuda")
        B.check(B.lib().turpy_plan_tune(plan.handle, B.TUNE_FORCE, ctypes.c_void_p(ws.data_ptr()), size,
                                        api._stream(), None, None))
        assert bool((ws[size:] == 0xA5).all())
        plan.close()


# 64 and 1024, one pair: every launch of the class runs one wave per transform,
# which takes no hint.  512, 4 pairs do too, but not the 7 of the same class
@pytest.mark.parametrize("n,r,classes", [(64, 4, []), (1024, 2, []), (256, 1, []), (512, 8, [3]), (512, 16, [4]),
                                         (2048, 1, [49]), (2048, 2, [1])])
def test_hints_where_a_launch_takes_one(api, n, r, classes):
    path = _path(n, r, 2)
    plan = api.Plan(path)
    u0 = torch.from_numpy(workloads.seeded_field((n, n), 9)).cuda()
    ref = plan.propagate(u0, seed=2)
    plan.set_config()
    plan.tune()
    for kernel in ("row_fwd", "row_bwd"):
        say(f"[tune] {kernel} n={n} R={r}: {_entry(api, kernel)}")
        assert [e["batch_class"] for e in _entry(api, kernel)] == classes
    cfg = plan.config
    plan.set_config(row_waves=cfg["row_waves"], row_waves_bwd=cfg["row_waves_bwd"])
    assert torch.equal(plan.propagate(u0, seed=2), ref)
    plan.close()


# above the one-wave line, so that the forward pass is the relay schedule and the
# adjoint the pair schedule; an odd count leaves the last pair's second half idle
@pytest.mark.parametrize("n,r", [(256, 34), (512, 11), (1024, 5)])
def test_hints_keep_the_bits_of_relay_and_pair(api, n, r):
    plan = api.Plan(_path(n, r, 2, 3))
    u0 = torch.from_numpy(workloads.seeded_field((n, n), 51)).cuda()
    g = torch.from_numpy(workloads.seeded_field((r, n, n), 52)).cuda()
    ref = plan.propagate(u0, seed=2)
    _, ck = plan.propagate(u0, seed=2, checkpoints=True)
    ref_in, ref_phi = plan.propagate_backward(g, ck, seed=2)
    for w in (2, 4):
        plan.set_config(row_waves=w, row_waves_bwd=w)
        assert torch.equal(plan.propagate(u0, seed=2), ref)
        g_in, g_phi = plan.propagate_backward(g, ck, seed=2)
        assert torch.equal(g_in, ref_in) and torch.equal(g_phi, ref_phi)
    plan.close()


# Untuned launches: the widest strip of which every CU has one (512: 8 columns,
# the AR step 16; 1024: 4 and 16).  One pair, ten screens at once; 1024 takes
# four screens of a pair to a launch, eight of a single realization
@pytest.mark.parametrize("n,r,m,synth,ar", [(512, 2, 10, 8, 16), (512, 2, 1, 4, 4), (512, 1, 10, 8, 16),
                                            (1024, 2, 8, 4, 16), (1024, 2, 1, 4, 4), (256, 2, 20, 16, 16)])
def test_reported_widths_are_the_launched_ones(api, n, r, m, synth, ar):
    plan = api.Plan(_path(n, r, m))
    cfg = plan.config
    assert (cfg["synth_width"], cfg["ar_width"]) == (synth, ar) and plan.widths["synth"] == synth
    plan.set_config(**cfg)
    assert plan.config == cfg
    plan.close()
