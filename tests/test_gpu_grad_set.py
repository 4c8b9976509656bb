"""Stored parameter gradients (gsr_project_bwd_set): whatever out held, they equal those accumulated into
zeros, value for value, with Gaussians in front of, beside and behind the cameras (rows without a gradient
are zero), for every SH degree, one and several views, and sizes around a workgroup of 256."""
import numpy as np
import pytest
import torch

from gpu_common import random_scene

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("deg", [0, 1, 2, 3])
@pytest.mark.parametrize("n,V", [(1, 1), (255, 1), (257, 2), (1024, 1), (3001, 3)])
def test_set_equals_accumulate_into_zeros(deg, n, V):
    import paper_2604_12942_amd as gsr
    G, cam = random_scene(n + deg, n, 64, 48, 50.0, sh_degree=deg, z_range=(-3.0, 6.0), xy_half=4.0)
    P = gsr.gaussians_to_device(G)
    ct = gsr.camera_tensor([cam] * V)
    r = gsr.Rasterizer(n, V, gsr.Raster(64, 48))
    r.forward(P, deg, ct)
    rng = np.random.default_rng(n)
    gC = torch.from_numpy(rng.standard_normal((V, 3, 48, 64)).astype(np.float32)).cuda()
    gD = torch.from_numpy(rng.standard_normal((V, 48, 64)).astype(np.float32)).cuda()
    r.render_backward(ct, gC, gD)
    out = []
    for accumulate in (True, False):
        grads = {k: torch.zeros_like(P[k]) if accumulate else torch.full_like(P[k], float("nan")) for k in gsr.PARAM_NAMES}
        gsr.project_bwd(P, deg, ct, V, r.raster, r.splats, r.dinst, r.em, r.tile_info, grads, r.dpose, r.pose_ws,
                        accumulate=accumulate)
        out.append((grads, r.dpose.clone()))
    seen = (r.tile_info.view(4, V, n)[0] > 0).any(0)
    assert n < 255 or (seen.any() and not seen.all())
    assert torch.equal(out[0][1], out[1][1])
    for k in gsr.PARAM_NAMES:
        assert torch.equal(out[0][0][k], out[1][0][k]), k
