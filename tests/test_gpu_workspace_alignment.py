"""Workspaces of the maintenance calls need no more than the alignment of the words they hold: at an odd multiple
of four bytes the results are those of an aligned one."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [3000, 140_000])
def test_maintenance_workspaces_at_four_bytes(n):
    import paper_2604_12942_amd as gsr
    g = torch.Generator("cuda").manual_seed(n)
    means = torch.rand(3, n, generator=g, device="cuda") * 20
    new = torch.rand(3, 500, generator=g, device="cuda") * 20
    logits = torch.randn(n, generator=g, device="cuda")
    seg = torch.randint(0, 5, (n,), generator=g, device="cuda", dtype=torch.int32)
    L = gsr.lib()
    big = torch.empty(max(L.gsr_row_order_workspace(n), L.gsr_prune_workspace(n), L.gsr_proximity_workspace(n, 500)) + 64,
                      dtype=torch.uint8, device="cuda")
    odd = big[4:]
    assert odd.data_ptr() % 8 == 4
    assert torch.equal(gsr.row_order(means, seg, ws=odd), gsr.row_order(means, seg))
    ka, kb = gsr.prune_select(logits, 0.0, 0.3, ws=odd), gsr.prune_select(logits, 0.0, 0.3)
    k = int(kb[1].item())
    assert int(ka[1].item()) == k and torch.equal(ka[0][:k], kb[0][:k])
    pa, pb = gsr.proximity_filter(means, new, 0.4, ws=odd), gsr.proximity_filter(means, new, 0.4)
    k = int(pb[2].item())
    assert torch.equal(pa[0], pb[0]) and int(pa[2].item()) == k and torch.equal(pa[1][:k], pb[1][:k])
