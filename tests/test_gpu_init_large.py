"""Voxel grouping of large clouds: runs of points that agree in the sorted hash bits longer than a lane's walk and
than a wave (crowded voxels, many points outside the grid), head counts scanned by a launch of their own (above
2^23 points) and 24 sorted hash bits (above 2^24).  Integers: equal to a sort by key, then whole hash."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _splitmix64(x):
    """SplitMix64 on int64 bit patterns."""
    def c(v):
        return v - (1 << 64) if v >> 63 else v

    def shr(z, k):
        return (z >> k) & ((1 << (64 - k)) - 1)
    z = x + c(0x9E3779B97F4A7C15)
    z = (z ^ shr(z, 30)) * c(0xBF58476D1CE4E5B9)
    z = (z ^ shr(z, 27)) * c(0x94D049BB133111EB)
    return z ^ shr(z, 31)


@pytest.mark.parametrize("n,crowd,outside", [(400_000, 0.9, 0.05), (1 << 21, 1.0, 0.0), ((1 << 23) + 9, 0.6, 0.3), ((1 << 24) + 7, 0.5, 0.1)])
def test_grouping_of_large_clouds(n, crowd, outside):
    import paper_2604_12942_amd as gsr
    g = torch.Generator("cuda").manual_seed(n)
    pts = torch.rand(3, n, generator=g, device="cuda")
    u = torch.rand(n, generator=g, device="cuda")
    pts *= torch.where(u < crowd, 0.49, 6.0)  # a part of them in one voxel, the others over some 1,700
    pts[0, u > 1.0 - outside] = 2000.0
    seed = 0x0123456789ABCDEF ^ n
    vox = gsr.voxel_pca(pts, seed)
    k = torch.floor(pts / 0.5).long()
    key = ((k[0] + 1024) << 21) | ((k[1] + 1024) << 10) | (k[2] + 511)
    key[pts[0] > 1000.0] = 0xFFFFFFFF
    h = _splitmix64(torch.arange(n, device="cuda") ^ seed)
    order = torch.sort(h ^ (-1 << 63), stable=True).indices
    order = order[torch.sort(key[order], stable=True).indices]
    assert torch.equal(vox["point_order"][:n].long(), order)
    uk, inv, cnt = torch.unique_consecutive(key[order], return_inverse=True, return_counts=True)
    nv = len(uk) - int((uk == 0xFFFFFFFF).sum())
    assert int(vox["n_voxels"].item()) == nv and int(vox["n_outside"].item()) == int((key == 0xFFFFFFFF).sum())
    pv = torch.empty(n, dtype=torch.long, device="cuda")
    pv[order] = torch.where(inv < nv, inv, -1)
    assert torch.equal(vox["point_voxel"][:n].long(), pv)
    start = torch.cumsum(cnt, 0) - cnt
    for name, ref in (("key", uk), ("start", start), ("count", cnt)):
        assert torch.equal(vox[name][:nv].long() & 0xFFFFFFFF, ref[:nv]), name
