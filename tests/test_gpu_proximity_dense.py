"""Proximity filter over crowded cells (up to thousands of map means in each): the lanes of a new mean stop
together once one has found a neighbour, and pairs of new means in one wave stop apart.  Decisions and indices
equal those of plain NumPy."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_map,spread", [(6000, 0.3), (6000, 1.0), (2000, 0.05)])
def test_proximity_in_crowded_cells(n_map, spread):
    import paper_2604_12942_amd as gsr
    rng = np.random.default_rng(n_map)
    d = 0.35
    A = rng.uniform(0, spread, (3, n_map)).astype(np.float32)
    # from inside the crowd out to two cells away, near and far ones next to each other
    B = rng.uniform(-2 * d, spread + 2 * d, (3, 1001)).astype(np.float32)
    B[:, ::3] = rng.uniform(0, spread, (3, 334)).astype(np.float32)
    keep, idx, n_keep = gsr.proximity_filter(torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda(), d)
    x = B.astype(np.float64)[:, :, None] - A.astype(np.float64)[:, None, :]
    want = ~(((x[0] * x[0] + x[1] * x[1]) + x[2] * x[2]) < float(np.float32(d)) ** 2).any(1)
    assert 0 < want.sum() < len(want)
    assert np.array_equal(keep[:1001].cpu().numpy().astype(bool), want)
    k = int(n_keep.item())
    assert k == want.sum() and np.array_equal(idx[:k].cpu().numpy(), np.nonzero(want)[0])
