"""Pair sums of more than 2^18 visible pairs take four lanes per pair where the first 64th of the list holds 16 records
per pair or more: both sides of that line, on pairs of up to 64 records, equal to a sequential float32 sum."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("VN,npairs,front", [(400_000, (1 << 18) + 1, 16), (400_000, (1 << 18) + 1, 15), (1 << 20, 1 << 20, 16),
                                             (1 << 20, 700_001, 64), ((1 << 20) + 1, 300_000, 40)])
def test_pair_sums_by_the_front_of_the_list(VN, npairs, front):
    import paper_2604_12942_amd as gsr
    g = torch.Generator("cuda").manual_seed(npairs + front)
    cnt = torch.randint(1, 5, (npairs,), generator=g, device="cuda")
    cnt[:npairs // 64] = front
    first = torch.cumsum(cnt, 0) - cnt
    M = int(cnt.sum())
    gid = torch.randperm(VN, generator=g, device="cuda")[:npairs]
    info = torch.zeros(4, VN, dtype=torch.int32, device="cuda")
    info[0, gid] = cnt.int()
    rec = torch.randn(M, 10, generator=g, device="cuda")
    pad = lambda x: torch.cat([x.int(), torch.zeros(VN - npairs, dtype=torch.int32, device="cuda")])
    pg, pf, np_, emit = pad(gid), pad(first), torch.tensor([npairs], dtype=torch.int32, device="cuda"), torch.zeros(M, dtype=torch.int32, device="cuda")
    out = torch.full((VN, 10), 3.0, device="cuda")
    gsr.pair_grads(rec, gsr.emission(emit, pg, pf, np_), info, VN, 1, out)
    want = torch.zeros(npairs, 10, device="cuda")
    for k in range(front if front > 4 else 4):
        at = torch.nonzero(cnt > k).flatten()
        want[at] += rec[first[at] + k]
    full = torch.zeros(VN, 10, device="cuda")
    full[gid] = want
    assert torch.equal(out, full)
