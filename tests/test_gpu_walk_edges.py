"""The forward walk of one 16x16 tile at the edges of its batches and groups: list lengths around 1, 64,
65, 128, 256 and 512 Gaussians (odd ones end on a null slot), faint (every pixel walks the whole list) and
opaque (pixels terminate on the first or the second of a pair, at every place of a group).  Images against the FP64 oracle with the gates and the knife-edge exclusion of the parity tests."""
import numpy as np
import pytest

import oracle

from gpu_common import KNIFE, img_close, random_scene, run_forward

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shift", [-4.0, 3.0])
@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 127, 129, 255, 256, 257, 511, 513])
def test_walk_matches_oracle(n, shift):
    G, cam = random_scene(n, n, 16, 16, 16.0, z_range=(2.0, 8.0), log_scale_mean=-0.5, xy_half=0.5, logit_shift=shift)
    for tile in ((16, 16), (8, 32), (32, 8)):
        out, rast, *_ = run_forward(G, [cam], tile=tile, sliced=False)
        o = oracle.render(G, cam)
        ok = o["margin"] >= KNIFE
        assert (~ok).sum() <= 0.05 * ok.size
        assert img_close(out["rgb"][0], o["rgb"], mask=np.broadcast_to(ok, o["rgb"].shape)).sum() == 0
        assert img_close(out["depth"][0], o["depth"], mask=ok).sum() == 0
        assert img_close(1 - out["T"][0], o["alpha"], mask=ok).sum() == 0
