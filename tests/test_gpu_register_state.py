"""register() with a state whose tensors were copied one by one (so that they no longer share one buffer), or that
holds only what gicp_iterate needs: the result is that of a state of its own, and the given tensors hold it."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("keep", ["clone", "needed"])
def test_register_with_a_copied_state(keep):
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
    want = loop.register(P, 0, seg, 1, cams, 1)
    assert want["iterations"] > 0 and not want["failed"]
    other = loop.register(P, 0, seg, 1, cams, 1, max_iter=3)["state"]
    state = {k: v.clone() if torch.is_tensor(v) else v for k, v in other.items()
             if keep == "clone" or k not in ("pose", "buf")}
    stats = state["stats"]
    for _ in range(2):
        got = loop.register(P, 0, seg, 1, cams, 1, state=state)
        for k in want:
            if k != "state":
                assert np.array_equal(got[k], want[k]), k
        assert torch.equal(stats, want["state"]["stats"]) and torch.equal(state["counts"], want["state"]["counts"])
