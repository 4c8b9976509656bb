"""More new means than one launch has lanes for (32 lanes each, fewer than 2^32 in a launch): 2^27 and a few.
They lie in a row a metre apart, each map mean within reach of the one it was put beside."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def test_more_new_means_than_a_launch_has_lane_groups():
    import paper_2604_12942_amd as gsr
    n = (1 << 27) + 11
    new = torch.zeros(3, n, device="cuda")
    j = torch.arange(n, device="cuda")
    new[0], new[1] = (j % 4096).float(), (j // 4096).float()  # exact in float32
    del j
    at = torch.tensor([0, 5, (1 << 23) - 1, 1 << 23, (1 << 26) + 3, (1 << 27) - 1, 1 << 27, n - 1], device="cuda")
    keep, idx, n_keep = gsr.proximity_filter((new[:, at] + 0.125).contiguous(), new, 0.25)
    assert int(n_keep.item()) == n - len(at)
    assert torch.equal(torch.nonzero(keep[:n] == 0).flatten(), at)
    left = torch.ones(n, dtype=torch.bool, device="cuda")
    left[at] = False
    assert torch.equal(idx[:n - len(at)], torch.nonzero(left).flatten().to(torch.int32))
