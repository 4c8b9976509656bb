"""Binning at the edges of its paths, on drawn tile rectangles and depth keys with many ties, against
numpy's lexicographic sort (integers: equal): one workgroup up to 8,192 pairs, block sums added up by
their readers up to 524,288, sorts of two launches per pass up to a capacity of 1M (1,024 keys a chunk up to
131,072 live ones, whole and partial chunks, kernels for 4 and 8 times that), 4 or 12 keys per thread
around a capacity of 4M, tile order in one workgroup up to 8,192 view-tiles, many view-tiles
with few pairs, no visible pair, and an overflow."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _draw(rng, VN, raster, visible, wide):
    on = rng.random(VN) < visible
    tx0, ty0 = rng.integers(0, raster.ntx, VN), rng.integers(0, raster.nty, VN)
    tx1 = np.minimum(tx0 + rng.integers(0, wide, VN), raster.ntx - 1)
    ty1 = np.minimum(ty0 + rng.integers(0, wide, VN), raster.nty - 1)
    nt = np.where(on, (tx1 - tx0 + 1) * (ty1 - ty0 + 1), 0)
    # depth keys of few distinct values, the sign bit set in some (a negative near plane)
    z = np.round(rng.uniform(-2, 20, VN) * 8).astype(np.float32).view(np.uint32)
    info = np.stack([nt, z, tx0 | ty0 << 16, tx1 | ty1 << 16]).astype(np.uint32)
    return info, nt, z, tx0, ty0, tx1


@pytest.mark.parametrize("n,V,size,cap,visible,wide", [
    (1, 1, (64, 48), 100, 1.0, 2), (8192, 1, (320, 240), 1 << 16, 0.9, 3), (8193, 1, (320, 240), 1 << 16, 0.9, 3),
    (2731, 3, (333, 211), 65_537, 0.5, 4), (5000, 2, (160, 120), 1 << 15, 0.0, 3), (3000, 4, (4096, 2048), 1 << 16, 0.5, 3),
    (300_000, 1, (1280, 720), 1_200_000, 0.3, 5), (524_288, 1, (640, 360), (1 << 22), 0.2, 4),
    (524_289, 1, (640, 360), (1 << 22) + 1, 0.2, 4), (175_000, 3, (1921, 1081), 1 << 20, 0.1, 5), (4000, 1, (320, 240), 5000, 1.0, 4),
    (131_072, 1, (640, 360), 1 << 17, 1.0, 1), (131_073, 1, (640, 360), 1 << 19, 1.0, 1),
    (524_287, 1, (640, 360), (1 << 19) + 1, 1.0, 1), (130_000, 4, (640, 360), 1 << 20, 0.85, 2),
    (150_000, 7, (640, 360), 1 << 20, 0.99, 1), (150_000, 7, (640, 360), (1 << 20) + 1, 0.99, 1)])
def test_binning_paths_match_lexsort(n, V, size, cap, visible, wide):
    import paper_2604_12942_amd as gsr
    rng = np.random.default_rng(n + V + cap)
    raster = gsr.Raster(*size, 16, 16)
    VN, T = V * n, raster.tiles
    info, nt, z, tx0, ty0, tx1 = _draw(rng, VN, raster, visible, wide)
    dev = lambda k, fill=7: torch.full((max(1, k),), fill, dtype=torch.int32, device="cuda")
    ti = torch.from_numpy(info.view(np.int32)).cuda().contiguous()
    gid, emit, pg, pf, npairs = dev(cap), dev(cap), dev(VN), dev(VN), dev(1)
    ranges, order, ninst = dev(2 * V * T), dev(V * T), dev(1)
    ws = dev(gsr.bin_sort_workspace(n, V, cap, raster) // 4 + 1)
    em = gsr.emission(emit, pg, pf, npairs)
    gsr.bin_sort(ti, n, V, raster, gid, cap, ranges, ninst, ws, order, em)
    M = int(nt.sum())
    assert ninst.item() == M
    rg = ranges.cpu().numpy().reshape(-1, 2)
    vis = np.nonzero(nt)[0]
    if M > cap:  # an overflow empties the frame
        assert not rg.any() and npairs.item() == 0 and not ti[0].any().item()
        assert np.array_equal(order.cpu().numpy(), np.arange(V * T))
        return
    # pairs by (depth key, pair), their tiles row-major, instances stably by view-tile
    porder = vis[np.lexsort((vis, z[vis]))]
    cnt = nt[porder]
    first = np.cumsum(cnt) - cnt
    assert npairs.item() == len(vis)
    assert np.array_equal(pg[:len(vis)].cpu().numpy(), porder) and np.array_equal(pf[:len(vis)].cpu().numpy(), first)
    g = porder.repeat(cnt)
    local = np.arange(M) - first.repeat(cnt)
    w = (tx1 - tx0 + 1)[g]
    key = (g // n) * T + (ty0[g] + local // w) * raster.ntx + tx0[g] + local % w
    srt = np.argsort(key, kind="stable")
    assert np.array_equal(gid[:M].cpu().numpy(), g[srt]) and np.array_equal(emit[:M].cpu().numpy(), srt)
    c = np.bincount(key, minlength=V * T)
    end = np.cumsum(c)
    assert np.array_equal(rg[:, 1] - rg[:, 0], c) and np.array_equal(rg[c > 0, 1], end[c > 0])
    # longest first, to 1/16 of an octave, ties by index
    e = np.maximum(np.floor(np.log2(np.maximum(c, 1))).astype(np.int64), 0)
    m = np.where(e >= 4, c >> np.maximum(e - 4, 0), c << np.maximum(4 - e, 0)) & 15
    lpt = np.where(c == 0, 0, e * 16 + m)
    assert np.array_equal(order.cpu().numpy(), np.argsort(-lpt, kind="stable"))
