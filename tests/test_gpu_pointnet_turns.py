"""The training backward where a wave takes more than one turn (more than 64 voxels per CU), with the biases'
ordered sum: shares that divide the waves (512, 1,024), that do not (300), and more shares than LDS rows.

The gradient is a sum over the voxels with a target, so a launch over all of them equals the sum of launches over
three disjoint masks with 256 blocks, which leave the ordered sum out.  A voxel's data path is the same in all, so only FP32 summation order differs:
a lane adds up to 3 turns x 8 voxels x 16 rows, then at most 1,024 shares are added one after another,
a random walk of 6e-8 per addition: below 1e-5 of |g| + rms(g)."""
import numpy as np
import pytest
import torch

from oracle import pointnet_oracle as pn
from test_gpu_pointnet import ORDER

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def scene():
    import paper_2604_12942_amd as gsr
    rng = np.random.default_rng(17)
    nv = 64 * torch.cuda.get_device_properties(0).multi_processor_count * 2 + 141
    cnt = rng.integers(1, 5, nv)
    k = np.arange(nv).repeat(cnt)
    base = np.stack([k % 50, (k // 50) % 50, k // 2500], 1) * 0.5
    pts = (base + rng.uniform(0.02, 0.48, (len(k), 3)) * [1.0, 1.0, 0.3]).astype(np.float32)
    t = torch.from_numpy(np.ascontiguousarray(pts[rng.permutation(len(pts))].T)).cuda()
    n = len(pts)
    vox = gsr.voxel_pca(t, 3)
    assert int(vox["n_voxels"].item()) == nv
    W = pn.init_weights(5)
    for b in ("b1", "b2", "b3", "b4", "b5"):
        W[b] = (rng.standard_normal(W[b].shape) * 0.1).astype(np.float32)
    wt = torch.from_numpy(np.concatenate([W[q].ravel() for q in ORDER]).astype(np.float32)).cuda()
    A = rng.standard_normal((nv, 3, 3)) * 0.05
    cov = A @ np.transpose(A, (0, 2, 1)) + np.eye(3) * 1e-3
    cov6, o_t = np.zeros((6, n), np.float32), np.zeros(n, np.float32)
    cov6[:, :nv] = np.stack([cov[:, 0, 0], cov[:, 0, 1], cov[:, 0, 2], cov[:, 1, 1], cov[:, 1, 2], cov[:, 2, 2]])
    o_t[:nv] = rng.uniform(0.05, 0.95, nv)
    args = torch.from_numpy(cov6).cuda(), torch.from_numpy(o_t).cuda()

    def grad(mask, blocks):
        g = torch.full((gsr.pointnet_weight_count(),), 7.0, dtype=torch.float32, device="cuda")
        loss = torch.zeros(1, dtype=torch.float64, device="cuda")
        gsr.pointnet_backward(t, vox, wt, *args, mask, 1.0 / nv, g, loss, blocks=blocks)
        return g.cpu().numpy().astype(np.float64), loss.item()

    part = torch.from_numpy(rng.integers(0, 3, n).astype(np.uint8)).cuda()
    parts = [grad((part == c).to(torch.uint8), 256) for c in range(3)]
    return W, grad, sum(p[0] for p in parts), sum(p[1] for p in parts), sum(abs(p[1]) for p in parts)


@pytest.mark.parametrize("blocks", [300, 512, 1024])
def test_backward_adds_up_over_several_turns(scene, blocks):
    W, grad, ref, l_ref, l_abs = scene
    whole, loss = grad(None, blocks)
    again, _ = grad(None, blocks)
    assert np.array_equal(whole, again)  # a fixed order
    assert abs(loss - l_ref) <= 1e-11 * l_abs
    off = 0
    for q in ORDER:
        size = np.asarray(W[q]).size
        a, b = whole[off:off + size], ref[off:off + size]
        off += size
        assert np.all(np.abs(a - b) <= 1e-5 * (np.abs(b) + np.sqrt(np.mean(b * b)))), q
