"""turpy_propagate_static where its fixed array holds fewer screens at a time
than turpy_propagate's workspace does (the subharmonic coefficients of many
pairs and screens take the rest): the same bits as the workspace call, and
refused only where not even one screen fits."""
import pytest
import torch

from paper_2604_07248_amd import binding as B
from paper_2604_07248_amd import workloads

pytestmark = pytest.mark.gpu

ROOM = 64 << 20


# 16: one screen of two (16 MiB apiece) beside 33 MiB of coefficients; 64: seven
# of eight (4 MiB apiece) beside 32 MiB
@pytest.mark.parametrize("n,r,m", [(16, 16000, 17), (64, 256, 1024)])
def test_fewer_screens_at_a_time(gpu_lib, n, r, m):
    from paper_2604_07248_amd import api
    dx = 4e-3
    path = workloads.uniform_path(n, n * dx, 1e-6, min(0.5 * n * dx * dx / 1e-6 * m, 2000.0), m, 1e-16, 0.005, 20.0, 3,
                                  realizations=r)
    plan = api.Plan(path)
    assert B.workspace_size(plan.handle, B.OP_PROPAGATE) > ROOM
    u0 = torch.from_numpy(workloads.seeded_field((n, n), 3)).cuda()
    want = plan.propagate(u0, seed=4, t=2)
    got = torch.full_like(want, float("nan"))
    B.check(gpu_lib.turpy_propagate_static(plan.handle, 4, 2, api._ptr(u0), 0, B.SCREENS_SYNTH, None, api._ptr(got),
                                           None, api._stream()))
    assert torch.equal(got, want)
    plan.close()


def test_refused_where_no_screen_fits(gpu_lib):
    from paper_2604_07248_amd import api
    path = workloads.uniform_path(64, 0.256, 1e-6, 500.0, 1100, 1e-16, 0.005, 20.0, 3, realizations=440)
    plan = api.Plan(path)  # 220 pairs: 6.9 MiB of screen and 59.1 MiB of coefficients
    u0 = torch.zeros((64, 64), dtype=torch.complex64, device="cuda")
    out = torch.zeros((440, 64, 64), dtype=torch.complex64, device="cuda")
    st = gpu_lib.turpy_propagate_static(plan.handle, 4, 2, api._ptr(u0), 0, B.SCREENS_SYNTH, None, api._ptr(out), None,
                                        api._stream())
    assert st == B.E_WORKSPACE and "static array" in B.last_error()
    plan.close()
