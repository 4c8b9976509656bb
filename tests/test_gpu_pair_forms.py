"""Pair sums take four lanes per pair up to 2^18 visible pairs of at most 2^20: both forms at the line, on pairs of up
to 64 records, whose sums are added in order (equal to a sequential float32 sum)."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("VN,npairs", [(400_000, (1 << 18) - 3), (400_000, 1 << 18), (400_000, (1 << 18) + 1), (1 << 18, 1 << 18),
                                       (1 << 20, 1 << 18), ((1 << 20) + 1, 1 << 18)])
def test_pair_sums_by_visible_pairs(VN, npairs):
    import paper_2604_12942_amd as gsr
    g = torch.Generator("cuda").manual_seed(npairs)
    cnt = torch.randint(1, 9, (npairs,), generator=g, device="cuda")
    cnt[::1000] = torch.randint(1, 65, (len(cnt[::1000]),), generator=g, device="cuda")
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
    for k in range(int(cnt.max())):
        at = torch.nonzero(cnt > k).flatten()
        want[at] += rec[first[at] + k]
    full = torch.zeros(VN, 10, device="cuda")
    full[gid] = want
    assert torch.equal(out, full)
