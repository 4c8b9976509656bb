"""The training backward at the edges of its work split: voxel counts around a wave's eight and a
workgroup's 64, past one turn of the launch, with one workgroup, with too few rows for the ordered
bias sum and with enough.

The reference is the kernel itself on parts: the gradient is a sum over the voxels with a target, so
one launch over all of them equals the sum of launches over three disjoint masks, whatever the
launch's size (the oracle test holds each part).  The data path of a voxel does not depend on the
split, so only FP32 summation order differs: at most 700 x 32 terms, a random walk of 6e-8 per
addition, 1e-5 of |g| + rms(g)."""
import numpy as np
import pytest
import torch

from oracle import pointnet_oracle as pn
from test_gpu_pointnet import ORDER

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nv,blocks", [(1, 512), (8, 1), (9, 512), (64, 512), (65, 1), (200, 3), (700, 512)])
def test_backward_adds_up_at_the_edges(nv, blocks):
    import paper_2604_12942_amd as gsr
    rng = np.random.default_rng(nv * 1000 + blocks)
    cnt = rng.integers(1, 45, nv)
    k = np.arange(nv).repeat(cnt)
    base = np.stack([k % 9, (k // 9) % 9, k // 81], 1) * 0.5
    pts = (base + rng.uniform(0.02, 0.48, (len(k), 3)) * [1.0, 1.0, 0.3]).astype(np.float32)
    pts = pts[rng.permutation(len(pts))]
    t = torch.from_numpy(np.ascontiguousarray(pts.T)).cuda()
    n = len(pts)
    vox = gsr.voxel_pca(t, 3)
    assert int(vox["n_voxels"].item()) == nv
    W = pn.init_weights(nv)
    for b in ("b1", "b2", "b3", "b4", "b5"):
        W[b] = (rng.standard_normal(W[b].shape) * 0.1).astype(np.float32)
    wt = torch.from_numpy(np.concatenate([W[q].ravel() for q in ORDER]).astype(np.float32)).cuda()
    A = rng.standard_normal((nv, 3, 3)) * 0.05
    cov = A @ np.transpose(A, (0, 2, 1)) + np.eye(3) * 1e-3
    cov6, o_t = np.zeros((6, n), np.float32), np.zeros(n, np.float32)
    cov6[:, :nv] = np.stack([cov[:, 0, 0], cov[:, 0, 1], cov[:, 0, 2], cov[:, 1, 1], cov[:, 1, 2], cov[:, 2, 2]])
    o_t[:nv] = rng.uniform(0.05, 0.95, nv)
    args = torch.from_numpy(cov6).cuda(), torch.from_numpy(o_t).cuda()

    def grad(mask, nb):
        g = torch.full((gsr.pointnet_weight_count(),), 7.0, dtype=torch.float32, device="cuda")
        loss = torch.zeros(1, dtype=torch.float64, device="cuda")
        gsr.pointnet_backward(t, vox, wt, *args, mask, 1.0 / nv, g, loss, blocks=nb)
        return g.cpu().numpy().astype(np.float64), loss.item()

    whole, l_whole = grad(None, blocks)
    part = torch.from_numpy(rng.integers(0, 3, n).astype(np.uint8)).cuda()
    parts = [grad((part == c).to(torch.uint8), nb) for c, nb in ((0, 5), (1, 256), (2, 512))]
    ref, l_ref = sum(p[0] for p in parts), sum(p[1] for p in parts)
    assert np.abs(whole).max() > 0 and abs(l_whole - l_ref) <= 1e-12 * sum(abs(p[1]) for p in parts)
    off = 0
    for q in ORDER:
        size = np.asarray(W[q]).size
        a, b = whole[off:off + size], ref[off:off + size]
        off += size
        assert np.all(np.abs(a - b) <= 1e-5 * (np.abs(b) + np.sqrt(np.mean(b * b)))), q
