"""The LDS-poison check on the row schedules, strips and kernels that the small
cases of test_gpu_lds_poison.py do not reach: the test build, which fills every
LDS array with NaN before a kernel uses it, gives the product build's bits, all
of them finite."""
import os
import subprocess
import sys

import numpy as np
import pytest

from paper_2604_07248_amd import build

from gpu_helpers import say

pytestmark = pytest.mark.gpu

HERE = os.path.dirname(os.path.abspath(__file__))


def test_poisoned_lds_gives_the_same_bits_on_every_schedule(gpu_lib, tmp_path):
    if not os.path.exists(build.POISON_LIB):
        pytest.fail("libturpy_poison.so is not built (run __graft_entry__.build())")
    sys.path.insert(0, HERE)
    import lds_poison_schedules
    from paper_2604_07248_amd import api
    api.tune_cache_clear()
    ref = lds_poison_schedules.run_cases()
    out = str(tmp_path / "poison.npz")
    env = dict(os.environ, TURPY_LIBRARY=build.POISON_LIB)
    say("[poison] child process with the poison build")
    res = subprocess.run([sys.executable, "-u", os.path.join(HERE, "lds_poison_schedules.py"), out], env=env,
                         stdout=subprocess.PIPE, text=True, timeout=300)
    assert res.returncode == 0
    got = np.load(out)
    assert sorted(got.files) == sorted(ref)
    for name, want in ref.items():
        assert want.any(), f"{name}: not finite"
        assert np.array_equal(got[name], want), name
    say(f"[poison] {len(ref)} outputs bitwise equal")
