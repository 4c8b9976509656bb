"""The list of depth slices: one workgroup up to 8,192 view-tiles, count, scan and emission launches above.
The same view rendered alone (exactly 8,192 tiles) and twice in one call (16,384) goes through both, and its
images are the same bits; a view with one row of tiles more (8,320) is above the line by itself."""
import numpy as np
import pytest
import torch

from gpu_common import long_tile_scene, run_forward

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H", [1024, 1040])
def test_slice_lists_agree(H):
    G, cam = long_tile_scene(W=2048, H=H)
    a, ra, *_ = run_forward(G, [cam], sliced=True)
    b, rb, *_ = run_forward(G, [cam, cam], sliced=True)
    rg = ra.tile_ranges.cpu().numpy().view(np.uint32).astype(np.int64).reshape(-1, 2)
    assert len(rg) == 128 * (H // 16) and (rg[:, 1] - rg[:, 0] > 8192).sum() >= 2
    for k in ("rgb", "depth", "T", "last"):
        for v in range(2):
            assert np.array_equal(a[k][0], b[k][v]), (k, v)
