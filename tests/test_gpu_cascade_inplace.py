"""The cascade with the colours' buffer as one of its outputs: each point's colour is read before its other
parameters are written, so the results equal those of separate buffers."""
import ctypes as C

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sh_degree", [0, 1])
@pytest.mark.parametrize("name", ["log_scales", "quats", "sh"])
@pytest.mark.parametrize("nv", [3000, 24_000])  # without and with room for the table of voxel records
def test_colours_in_place_of_an_output(name, sh_degree, nv):
    import paper_2604_12942_amd as gsr
    from paper_2604_12942_amd import _abi
    rng = np.random.default_rng(7)
    per = 12
    n = nv * per
    c = np.arange(nv).repeat(per)
    base = np.stack([c % 20, (c // 20) % 20, c // 400], 1) * 0.5
    pts = (base + rng.uniform(0.05, 0.45, (n, 3)) * [1.0, 1.0, 0.1]).astype(np.float32)[rng.permutation(n)]
    t = torch.from_numpy(np.ascontiguousarray(pts.T)).cuda()
    col, dep = torch.rand(3, n, device="cuda"), 1.0 + 9.0 * torch.rand(n, device="cuda")
    vox = gsr.voxel_pca(t, 5)
    ref, b_ref = gsr.cascade(t, col, dep, vox, focal=320.0, sh_degree=sh_degree)
    P = {k: torch.empty_like(ref[k]) for k in gsr.PARAM_NAMES}
    P[name].view(-1)[:3 * n] = col.view(-1)
    branch = torch.empty_like(b_ref)
    ws = torch.empty(1024, dtype=torch.int32, device="cuda")
    p = lambda a: C.c_void_p(a.data_ptr())
    V = _abi.Voxels(*[p(vox[k]) for k in gsr.VOXEL_FIELDS])
    O = _abi.Params(*[p(P[k]) for k in gsr.PARAM_NAMES])
    assert gsr.lib().gsr_cascade(p(t), p(P[name]), p(dep), None, 0, n, C.byref(V), None, 320.0, 0.0, sh_degree, C.byref(O),
                                 p(branch), p(ws), ws.numel() * 4, C.c_void_p(torch.cuda.current_stream().cuda_stream)) == 0
    assert torch.equal(b_ref, branch)
    for k in gsr.PARAM_NAMES:
        assert torch.equal(ref[k], P[k]), k
