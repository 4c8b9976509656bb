"""The cascade's results do not depend on the voxel count: it is optional, and whatever it says (nothing, zero,
too few, too many), every parameter is the same bits, in small clouds and in those large enough for the table of
voxel records."""
import ctypes as C

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sh_degree", [0, 1])
@pytest.mark.parametrize("anchored", [False, True])
@pytest.mark.parametrize("nv,model", [(500, True), (12_000, True), (12_000, False), (24_000, False)])
def test_cascade_does_not_depend_on_the_voxel_count(sh_degree, anchored, nv, model):
    import paper_2604_12942_amd as gsr
    from paper_2604_12942_amd import _abi
    rng = np.random.default_rng(31)
    per = 12
    n = nv * per
    c = np.arange(nv).repeat(per)
    base = np.stack([c % 30, (c // 30) % 30, c // 900], 1) * 0.5
    pts = (base + rng.uniform(0.05, 0.45, (n, 3)) * [1.0, 1.0, 0.1]).astype(np.float32)[rng.permutation(n)]
    pts[:5] = 2000.0  # outside the grid
    t = torch.from_numpy(np.ascontiguousarray(pts.T)).cuda()
    col, dep = torch.rand(3, n, device="cuda"), 1.0 + 9.0 * torch.rand(n, device="cuda")
    seg = torch.from_numpy(rng.integers(0, 3, n).astype(np.int32)).cuda()
    pred = torch.from_numpy(rng.normal(-3.0, 1.5, (8, n)).astype(np.float32)).cuda()
    vox = gsr.voxel_pca(t, 5)
    assert int(vox["n_voxels"].item()) == nv
    ws = torch.empty(1024, dtype=torch.int32, device="cuda")
    fn = gsr.lib().gsr_cascade_anchored if anchored else gsr.lib().gsr_cascade
    p = lambda a: C.c_void_p(a.data_ptr())

    def run(count):
        K = (sh_degree + 1) ** 2
        P = {k: torch.full((r, n), float("nan"), device="cuda") for k, r in
             (("means", 3), ("log_scales", 3), ("quats", 4), ("opacity_logits", 1), ("sh", 3 * K))}
        branch = torch.full((n,), 9, dtype=torch.uint8, device="cuda")
        V = _abi.Voxels(*[p(vox[k]) for k in gsr.VOXEL_FIELDS])
        held = None if count is None else torch.from_numpy(np.array([count], np.uint32).view(np.int32)).cuda()
        V.n_voxels = None if held is None else held.data_ptr()
        O = _abi.Params(*[p(P[k]) for k in gsr.PARAM_NAMES])
        assert fn(p(t), p(col), p(dep), p(seg), 3, n, C.byref(V), p(pred) if model else None, 320.0, 0.0, sh_degree, C.byref(O), p(branch),
                  p(ws), ws.numel() * 4, C.c_void_p(torch.cuda.current_stream().cuda_stream)) == 0
        torch.cuda.synchronize()
        return P, branch

    P, b = run(nv)
    assert sorted(b.unique().tolist()) == ([0, 1, 2] if model else [1, 2])
    for count in (None, 0, 1, nv - 1, nv + 7, n, n + 1, 0xFFFFFFFF):
        Q, bq = run(count)
        assert torch.equal(b, bq), count
        for k in P:
            assert torch.equal(P[k], Q[k]), (count, k)
