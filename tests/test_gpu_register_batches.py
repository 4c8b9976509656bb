"""register() queues its iterations in batches (8, then as many again): its result equals that of the same
iterations queued at once, for iteration limits below, at and above the batches' ends, with a state of its
own and with one used again."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("max_iter", [0, 1, 7, 8, 9, 16, 17, 30])
def test_batches_equal_one_queue(max_iter):
    import paper_2604_12942_amd as gsr
    import synth
    from paper_2604_12942_amd import loop
    rng = np.random.default_rng(3)
    n = 3000
    base = rng.uniform(-3, 3, (3, n)).astype(np.float32)
    base[2] = 0.3 * np.sin(base[0]) + 0.2 * np.cos(2 * base[1]) + 5
    means = np.concatenate([base, base + np.array([[0.08], [-0.05], [0.04]], np.float32)], axis=1)
    g = dict(means=means, log_scales=np.full((3, 2 * n), -3.0, np.float32),
             quats=np.tile(np.array([[1], [0], [0], [0]], np.float32), (1, 2 * n)),
             opacity_logits=np.zeros(2 * n, np.float32), sh=np.zeros((3, 2 * n), np.float32), sh_degree=0)
    P = gsr.gaussians_to_device(g)
    seg = torch.from_numpy(np.repeat(np.array([0, 1], np.int32), n)).cuda()
    cams = gsr.camera_tensor([synth.make_camera(np.eye(3), np.zeros(3), 60.0, 60.0, 32.0, 32.0, 64, 64)])
    st = gsr.gicp_prepare(P, 0, seg, 1, cams, 1, 30.0, 0.5)
    pose = torch.tensor([1.0, 0, 0, 0, 1, 0, 0, 0, 1, 0, 0, 0], dtype=torch.float64, device="cuda")
    gsr.gicp_iterate(P, 0, st, pose, max_iter)
    want, ws = pose.cpu().numpy(), st["stats"].cpu().numpy()
    state = None
    for _ in range(2):
        r = loop.register(P, 0, seg, 1, cams, 1, max_iter=max_iter, state=state)
        state = r["state"]
        assert np.array_equal(np.append(r["R"].ravel(), r["t"]), want)
        assert r["iterations"] == int(ws[37]) <= max_iter and r["converged"] == bool(ws[36])
        assert r["cost"] == ws[27] and r["count"] == int(ws[29]) and not r["failed"]
        assert [r["n_src"], r["n_tgt"]] == st["counts"].cpu().tolist()
