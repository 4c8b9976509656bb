"""Branches of the voxel grouping and of the cascade: points of one voxel that agree in the sorted hash
bits (crowded voxels), blocks of 1,024 and 4,096 points, points outside the grid; the cascade's voxel
table against its per-point form.  Integers and copies: equal."""
import ctypes as C

import numpy as np
import pytest
import torch

from oracle import init_oracle as io

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,extent", [(1, 0.2), (1023, 0.2), (60_000, 0.45), (300_000, 1.4), ((1 << 20) + 5, 6.0)])
def test_point_order_is_by_key_then_whole_hash(n, extent):
    import paper_2604_12942_amd as gsr
    rng = np.random.default_rng(n)
    pts = rng.uniform(0.0, extent, (n, 3)).astype(np.float32)
    pts[rng.random(n) < 0.001] = 2000.0  # outside the grid
    seed = 0x9E3779B97F4A7C15 ^ n
    vox = gsr.voxel_pca(torch.from_numpy(np.ascontiguousarray(pts.T)).cuda(), seed)
    k = np.floor(pts.astype(np.float64) / 0.5).astype(np.int64)
    out = pts[:, 0] > 1000.0
    key = np.where(out, 0xFFFFFFFF, ((k[:, 0] + 1024) << 21) | ((k[:, 1] + 1024) << 10) | (k[:, 2] + 511))
    h = io.splitmix64(np.uint64(seed) ^ np.arange(n, dtype=np.uint64))
    order = np.lexsort((h, key))
    assert np.array_equal(vox["point_order"].cpu().numpy()[:n], order)
    assert int(vox["n_outside"].item()) == out.sum()
    uk, start, inv, cnt = np.unique(key[order], return_index=True, return_inverse=True, return_counts=True)
    nv = len(uk) - (1 if out.any() else 0)
    assert int(vox["n_voxels"].item()) == nv
    pv = np.empty(n, np.int64)
    pv[order] = np.where(inv < nv, inv, 0xFFFFFFFF)
    assert np.array_equal(vox["point_voxel"].cpu().numpy().view(np.uint32)[:n], pv.astype(np.uint32))
    for name, ref in (("key", uk), ("start", start), ("count", cnt)):
        assert np.array_equal(vox[name].cpu().numpy().view(np.uint32)[:nv], ref[:nv].astype(np.uint32)), name


@pytest.mark.parametrize("per_voxel", [1, 2, 3, 12])
@pytest.mark.parametrize("anchored", [False, True])
def test_cascade_table_equals_per_point_form(per_voxel, anchored):
    """SH degree 1 has room for the table at any density, degree 0 only above 2.75 points per voxel, and
    colours converted in place leave none: all three agree, and the branches are the oracle's."""
    import paper_2604_12942_amd as gsr
    from paper_2604_12942_amd import _abi
    rng = np.random.default_rng(per_voxel)
    nv, n = 700, 700 * per_voxel
    c = np.arange(nv).repeat(per_voxel)
    base = np.stack([c % 9, (c // 9) % 9, c // 81], 1) * 0.5
    pts = (base + rng.uniform(0.05, 0.45, (n, 3)) * [1.0, 1.0, 0.1]).astype(np.float32)[rng.permutation(n)]
    pts[:3] = 2000.0
    t = torch.from_numpy(np.ascontiguousarray(pts.T)).cuda()
    col, dep = torch.rand(3, n, device="cuda"), 1.0 + 9.0 * torch.rand(n, device="cuda")
    seg = torch.from_numpy(rng.integers(0, 3, n).astype(np.int32)).cuda()
    vox = gsr.voxel_pca(t, 5)
    pred = torch.from_numpy(rng.normal(-3.0, 1.5, (8, n)).astype(np.float32)).cuda()
    pred[0, ::7] = float("nan")
    kw = dict(pred=pred, focal=320.0, segment=seg, n_segments=3, anchored=anchored)
    P0, b0 = gsr.cascade(t, col, dep, vox, sh_degree=0, **kw)
    P1, b1 = gsr.cascade(t, col, dep, vox, sh_degree=1, **kw)
    P2 = {k: torch.empty_like(P0[k]) for k in P0}
    b2, col2 = torch.empty_like(b0), col.clone()
    P2["sh"] = col2
    ws = torch.empty(1024, dtype=torch.int32, device="cuda")
    V = _abi.Voxels(*[C.c_void_p(vox[k].data_ptr()) for k in gsr.VOXEL_FIELDS])
    O = _abi.Params(*[C.c_void_p(P2[k].data_ptr()) for k in gsr.PARAM_NAMES])
    fn = gsr.lib().gsr_cascade_anchored if anchored else gsr.lib().gsr_cascade
    p = lambda a: C.c_void_p(a.data_ptr())
    assert fn(p(t), p(col2), p(dep), p(seg), 3, n, C.byref(V), p(pred), 320.0, 0.0, 0, C.byref(O), p(b2), p(ws), ws.numel() * 4,
              C.c_void_p(torch.cuda.current_stream().cuda_stream)) == 0
    for P, b in ((P1, b1), (P2, b2)):
        assert torch.equal(b0, b)
        for k in gsr.PARAM_NAMES:
            assert torch.equal(P0[k], P[k][:3] if k == "sh" else P[k]), k
    assert not P1["sh"][3:].any().item()
    pv = vox["point_voxel"].cpu().numpy().view(np.uint32).astype(np.int64)
    inside = pv != 0xFFFFFFFF
    pv[~inside] = 0
    valid = io.prediction_valid(pred.cpu().numpy().T)[pv] & inside
    rel = vox["reliable"].cpu().numpy()[pv].astype(bool) & inside
    assert np.array_equal(b0.cpu().numpy(), np.where(valid, 0, np.where(rel, 1, 2)))
