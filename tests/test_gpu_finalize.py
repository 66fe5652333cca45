"""The statistics' finalize call over many blocks (with an SI map to hold the
partial sums) against the one-block form (no map) and the FP64 oracle, at grid
sizes around the block split: 64 is the smallest that takes it, 100 and 257
are not powers of two (a last block partly full), 1024 gives every block
several pixels per thread, and 63 stays with one block."""
import numpy as np
import pytest
import torch

from oracle import stats as ost
from paper_2604_07248_amd import binding as B

pytestmark = pytest.mark.gpu


def _finalize(buf, n, dx, count, weight, fraction, with_map):
    from paper_2604_07248_amd import api
    si = torch.full((n, n), -7.0, dtype=torch.float32, device="cuda") if with_map else None
    out = torch.empty(8, dtype=torch.float64, device="cuda")
    B.stats(n, dx, 0, None, api._ptr(buf), count, 1, api._ptr(si), api._ptr(out), api._stream(), api._ptr(weight),
            fraction)
    return si, out.cpu().numpy()


@pytest.mark.parametrize("n", [16, 63, 64, 100, 128, 257, 1024])
@pytest.mark.parametrize("fraction", [0.0, 0.5, 0.999, 1.0])
def test_many_blocks_equal_one_block(gpu_lib, n, fraction):
    rng = np.random.default_rng(n)
    dx, count = 0.003, 7
    x = (np.arange(n) - n // 2) * dx
    r2 = x[None, :] ** 2 + x[:, None] ** 2
    inten = np.exp(-2 * r2 / (0.15 * n * dx) ** 2)[None] * rng.exponential(size=(count, n, n))
    buf = np.zeros((4, n, n), dtype=np.float32)
    buf[0] = inten.sum(0)
    buf[1] = 1e-8 * buf[0] * rng.standard_normal((n, n))
    buf[2] = (inten ** 2).sum(0)
    dev = torch.from_numpy(buf).cuda()
    weight = torch.from_numpy((r2 <= (0.3 * n * dx) ** 2).astype(np.float32)).cuda()
    si, many = _finalize(dev, n, dx, count, weight, fraction, True)
    again, many2 = _finalize(dev, n, dx, count, weight, fraction, True)
    _, one = _finalize(dev, n, dx, count, weight, fraction, False)
    assert np.array_equal(many, many2) and torch.equal(si, again)
    b = buf.astype(np.float64)
    m1, m2 = (b[0] - b[1]) / count, (b[2] - b[3]) / count
    m1f = m1.astype(np.float32)
    if fraction == 1.0:
        # Every pixel belongs to a region that holds all of the power, as far as the FP64 total (whose order
        # the two forms do not share) can tell: what lies below the threshold is lost in the total's rounding.
        for thr in (many[6], one[6]):
            assert m1f[m1f < thr].astype(np.float64).sum() <= m1f.size * 2.0 ** -53 * m1f.sum(dtype=np.float64)
        same = [1, 2, 3, 7]
    else:
        assert many[6] == one[6] and many[5] == one[5] and many[3] == count
        same = list(range(8))
    if 0 < fraction < 1:
        assert many[6] == ost.power_cutoff_threshold(m1f, fraction)
    # FP64 sums of up to 2^20 terms in another order: 2^20 * 2^-53 at most
    assert np.all(np.abs(many - one)[same] <= 2.0 ** -33 * np.abs(one)[same])
    with np.errstate(divide="ignore", invalid="ignore"):
        ref = (m2 / (m1 * m1) - 1.0).astype(np.float32)
    assert np.array_equal(si.cpu().numpy(), ref)
