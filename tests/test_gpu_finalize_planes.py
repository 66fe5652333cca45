"""The statistics' finalize call on the largest grid it takes, n = 65536: 2^32
pixels, more than a launch may have threads in x.  The moments are those of a
constant intensity of known mean square, exact in FP32, but for a few brighter
pixels, so every output is known; the map holds other values before."""
import math

import pytest
import torch

from paper_2604_07248_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fraction", [0.0, 1e-9])
def test_largest_grid(gpu_lib, fraction):
    if torch.cuda.mem_get_info()[0] < 150e9:
        pytest.skip("needs 86 GB of free device memory")
    n, count = 1 << 16, 2
    at = torch.tensor([5, 2 ** 31 + 1, 2 ** 32 - 300, 2 ** 32 - 1], device="cuda")
    buf = torch.zeros((4, n, n), device="cuda")
    buf[0], buf[2] = 4.0, 10.0                              # mean 2, mean square 5: SI = 1/4
    buf[0].view(-1)[at], buf[2].view(-1)[at] = 8.0, 64.0    # mean 4, mean square 32: SI = 1
    si = torch.full((n, n), -7.0, device="cuda")
    out = torch.zeros(8, dtype=torch.float64, device="cuda")
    p = lambda t: t.data_ptr()  # noqa: E731
    B.stats(n, 1e-3, 0, None, p(buf), count, 1, p(si), p(out), torch.cuda.current_stream().cuda_stream, None, fraction)
    s = out.cpu().tolist()
    assert bool((si.view(-1)[at] == 1.0).all())
    assert int(torch.count_nonzero(si == 0.25)) == n * n - len(at)
    if fraction == 0.0:
        region = (n // 2 - 1) ** 2      # |i - n/2| < n/4; the bright pixel 2^31 + 1 lies outside it
        assert s[5] == region and s[4] == 0.25 * region and s[0] == 0.25 and s[6] == 0.0
    else:                               # the four bright pixels hold 16 of 2^33 + 8
        assert 16 / (2 ** 33 + 8) > fraction and s[6] == 4.0 and s[5] == 4 and s[0] == 1.0
    mean_r2 = 2 * 1e-6 * sum((i - n // 2) ** 2 for i in range(n)) / n
    assert math.isclose(s[1], math.sqrt(2 * mean_r2), rel_tol=1e-6) and s[3] == count
    del buf, si
    torch.cuda.empty_cache()
