"""Pair sums at the edges of their split: four lanes per pair up to 1M (view, Gaussian) pairs, one lane
above; whole and partial waves of 16 and 64 pairs; pairs of up to 64 records (added in order: equal to a
sequential float32 sum) and above (64 strided partial sums and a tree of 6 levels: n records differ from
the float64 sum by at most (n/64 + 6) rounding steps of the sum of magnitudes)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("VN", [1 << 20, (1 << 20) + 1])
@pytest.mark.parametrize("npairs", [0, 1, 15, 16, 17, 63, 64, 65, 255, 256, 257, 5000])
def test_pair_sums_at_the_split(VN, npairs):
    import paper_2604_12942_amd as gsr
    rng = np.random.default_rng(npairs)
    cnt = rng.choice([1, 2, 7, 31, 63, 64, 65, 300, 1025], max(npairs, 1))[:npairs]
    first = np.cumsum(cnt) - cnt
    M = int(cnt.sum())
    gid = rng.permutation(VN)[:npairs]
    ntiles = np.zeros(4 * VN, np.int32)
    ntiles[gid] = cnt
    rec = rng.standard_normal((max(M, 1), 10)).astype(np.float32)
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()
    pad = lambda x: dev(np.append(x, [0] * (VN - npairs)).astype(np.int32))
    pg, pf, np_, ti, dinst = pad(gid), pad(first), dev(np.array([npairs], np.int32)), dev(ntiles), dev(rec)
    emit = torch.zeros(max(M, 1), dtype=torch.int32, device="cuda")
    out = torch.full((VN, 10), 3.0, device="cuda")
    gsr.pair_grads(dinst, gsr.emission(emit, pg, pf, np_), ti, VN, 1, out)
    got = out.cpu().numpy()
    rest = np.ones(VN, bool)
    rest[gid] = False
    assert not got[rest].any()
    for q in range(npairs):
        part = rec[first[q]:first[q] + cnt[q]]
        if cnt[q] <= 64:
            acc = np.zeros(10, np.float32)
            for r in part:
                acc += r
            assert np.array_equal(got[gid[q]], acc), q
        else:
            p = part.astype(np.float64)
            assert np.all(np.abs(got[gid[q]] - p.sum(0)) <= (cnt[q] / 64 + 7) * 6e-8 * np.abs(p).sum(0)), q
