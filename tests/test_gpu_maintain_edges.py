"""Proximity filter and row order at the sizes where their splits can go wrong: one 32-lane group per new mean,
eight to a workgroup; the scan's 16 consecutive words per thread and 4,096 per workgroup; the bounding box over
one, a few and 256 partials.  Decisions and indices equal those of plain NumPy."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_new", [1, 7, 8, 9, 15, 16, 17, 255, 257, 4095, 4096, 4097])
@pytest.mark.parametrize("n_map", [1, 33, 1000])
def test_proximity_edges(n_new, n_map):
    import paper_2604_12942_amd as gsr
    rng = np.random.default_rng(n_new + n_map)
    d = 0.4
    A = rng.uniform(-2, 2, (3, n_map)).astype(np.float32)
    B = rng.uniform(-2, 2, (3, n_new)).astype(np.float32)
    keep, idx, n_keep = gsr.proximity_filter(torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda(), d)
    x = B.astype(np.float64)[:, :, None] - A.astype(np.float64)[:, None, :]
    dd = float(np.float32(d)) ** 2
    want = ~(((x[0] * x[0] + x[1] * x[1]) + x[2] * x[2]) < dd).any(1)
    assert np.array_equal(keep[:n_new].cpu().numpy().astype(bool), want)
    k = int(n_keep.item())
    assert k == want.sum() and np.array_equal(idx[:k].cpu().numpy(), np.nonzero(want)[0])


@pytest.mark.parametrize("n", [1, 64, 255, 257, 16_385, 70_001])
def test_row_order_edges(n):
    import paper_2604_12942_amd as gsr
    rng = np.random.default_rng(n)
    m = rng.uniform(-40, 60, (3, n)).astype(np.float32)
    m[:, -1] = 70.0  # the box's far corner in the last row
    got = gsr.row_order(torch.from_numpy(m).cuda())[:n].cpu().numpy().view(np.uint32).astype(np.int64)
    lo, hi = m.min(1), m.max(1)
    code = np.zeros(n, np.uint64)
    for a in range(3):
        sc = np.float32(1024.0) / (hi[a] - lo[a]) if hi[a] > lo[a] else np.float32(0)
        q = np.clip(np.floor((m[a] - lo[a]) * sc), 0, 1023).astype(np.uint64)
        for b in range(10):
            code |= (q >> np.uint64(b) & np.uint64(1)) << np.uint64(3 * b + a)
    assert np.array_equal(got, np.argsort(code, kind="stable"))
