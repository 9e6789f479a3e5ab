"""Selection from candidate windows on both sides of the number of roots from which eight lanes serve a root."""
import numpy as np
import pytest
import torch

import oracle
import paper_2402_05396_amd as T


@pytest.mark.gpu
@pytest.mark.parametrize("roots", [7999, 8000, 8001, 8007, 8032])
@pytest.mark.parametrize("m,k", [(16, 10), (17, 1), (17, 16), (25, 8), (25, 9), (32, 31), (32, 32), (33, 10), (64, 63), (64, 17)])
@pytest.mark.parametrize("large", [0, 7, 1])
def test_matches_the_oracle(roots, m, k, large):
    """large: every how many roots have weights that need 64-bit sums (0: none)."""
    rng = np.random.default_rng(roots + 97 * m + k)
    weight = rng.integers(1, 1 << 26, (roots, m), dtype=np.uint64).astype(np.uint32)
    if large:
        weight[::large] = rng.integers(1, 1 << 32, (len(weight[::large]), m), dtype=np.uint64).astype(np.uint32)
        weight[::5 * large] = 0xFFFFFFFF
    weight[3::11] = 1
    weight[4::13, m // 2] = (1 << 26) - 1
    count = rng.integers(0, m + 1, roots).astype(np.int32)
    count[::2], count[5::17], count[6::19], count[7::23] = m, m + 3, -2, k
    dev = lambda a: torch.from_numpy(a).cuda()
    cand = dict(nbr=dev(rng.integers(0, 1 << 30, (roots, m)).astype(np.int32)), eid=dev(rng.integers(0, 1 << 30, (roots, m)).astype(np.int32)),
                ts=dev(rng.integers(-(1 << 60), 1 << 60, (roots, m))))
    want_sel, want_count = oracle.select_weighted(weight, np.clip(count, 0, m), k, seed=5, hop=3)
    sel, got_count, kept = T.select_weighted(dev(weight.view(np.int32)), dev(count), k, 5, 3, candidates=cand)
    assert np.array_equal(sel.cpu().numpy(), want_sel) and np.array_equal(got_count.cpu().numpy(), want_count)
    at = torch.from_numpy(want_sel).cuda().long()
    for f, pad in (("nbr", -1), ("eid", -1), ("ts", 0)):
        assert torch.equal(kept[f], torch.where(at >= 0, cand[f].gather(1, at.clamp(min=0)), torch.full_like(cand[f][:, :1], pad))), f
