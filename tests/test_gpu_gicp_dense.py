"""The registration's search in crowded cells, where candidates are reached through boxes of 256 and of 16: cells of
64 targets (the largest scanned one by one), 65, 257 and more than 4,096 (a second turn over the boxes of 256), runs
that begin and end inside boxes, targets on a lattice and sources half a step beside it (equal distances within and
across boxes), the same target many times over, sources at about the search radius, and buckets of many small
cells.  Correspondences are integers: equal."""
import numpy as np
import pytest
import torch

import synth
from oracle import gicp_oracle as go

pytestmark = pytest.mark.gpu

CELL = 0.5  # the search radius, and within a millionth the cells' edge


def _check(tgt, src, d_corr, seed):
    import paper_2604_12942_amd as gsr
    rng = np.random.default_rng(seed)
    n = len(tgt) + len(src)
    g = synth.random_gaussians(seed, n, 0)
    perm = rng.permutation(n)  # list positions unrelated to the places
    seg = np.concatenate([np.zeros(len(tgt)), np.ones(len(src))]).astype(np.int32)[perm]
    g["means"] = np.ascontiguousarray(np.concatenate([tgt, src])[perm].T.astype(np.float32))
    cam = synth.make_camera(np.eye(3), np.zeros(3), 20.0, 20.0, 500.0, 500.0, 1000, 1000)
    P = gsr.gaussians_to_device(g)
    st = gsr.gicp_prepare(P, 0, torch.from_numpy(seg).cuda(), 1, gsr.camera_tensor([cam]), 1, 1000.0, d_corr)
    assert st["counts"].cpu().tolist() == [len(src), len(tgt)]
    pose = torch.tensor([1.0, 0, 0, 0, 1, 0, 0, 0, 1, 0, 0, 0], dtype=torch.float64, device="cuda")
    corr = torch.full((n,), -7, dtype=torch.int32, device="cuda")
    gsr.gicp_iterate(P, 0, st, pose, 1, corr=corr)
    m = g["means"].astype(np.float64)
    ref = go.correspondences(m[:, seg == 1], m[:, seg == 0], d_corr)
    assert (ref >= 0).any() and (ref < 0).any()
    assert np.array_equal(corr[:len(src)].cpu().numpy(), ref)


def _cells(rng, counts, step):
    """counts[k] targets on the lattice of the given step in the k-th of a row of cells around (0, 0, 6)."""
    side = int(CELL / step)
    out = []
    for k, c in enumerate(counts):
        q = rng.integers(0, side, (c, 3)) * step
        out.append(q + [CELL * (k - 2) + 1e-3, 1e-3, 6.0 + 1e-3])
    return np.concatenate(out)


@pytest.mark.parametrize("counts", [[64], [65], [257], [5000], [5, 70, 300, 1000, 4200], [63, 66, 15, 17, 260], [1, 4097, 1]])
@pytest.mark.parametrize("step", [1 / 32, 1 / 8])
def test_crowded_cells(counts, step):
    rng = np.random.default_rng(sum(counts) + int(1 / step))
    tgt = _cells(rng, counts, step)
    lo, hi = tgt.min(0) - 0.7, tgt.max(0) + 0.7
    src = lo + np.round(rng.uniform(0, 1, (400, 3)) * (hi - lo) / step) * step + step / 2
    _check(tgt, src, CELL, len(tgt))


@pytest.mark.parametrize("n", [64, 65, 300, 4500])
def test_the_same_target_many_times(n):
    rng = np.random.default_rng(n)
    tgt = np.tile([[0.125, 0.25, 6.125]], (n, 1))
    tgt[n // 2:] += [0.0, 0.0, 0.25]
    src = np.array([0.125, 0.25, 6.25]) + rng.integers(-6, 7, (300, 3)) * 0.125
    _check(tgt, src, CELL, n)


def test_buckets_of_many_cells():
    rng = np.random.default_rng(5)
    tgt = rng.uniform(-20, 20, (400_000, 3)) + [0, 0, 60.0]  # cells of 2 cm, six to a bucket, a target in each
    src = tgt[rng.integers(0, len(tgt), 300)] + rng.normal(0, 0.012, (300, 3))
    _check(tgt, src, 0.02, 5)
