"""Draws with 1, 2, 64 and 65 sums of the selector's top level, which decide what is read before the random number is known."""
import numpy as np
import pytest
import torch

import oracle
import paper_2402_05396_amd as T

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1 << 20, (1 << 20) + 1, 64 << 20, (64 << 20) + 1])
def test_draws(n):
    rng = np.random.default_rng(n % 1000)
    score = rng.integers(0, 1 << 32, n, dtype=np.uint64).astype(np.uint32)
    score[: n // 2] = 0                      # the first sums of every level are 0
    score[-1] = 0xFFFFFFFF
    s = T.selector_init(torch.from_numpy(score.view(np.int32)).cuda())
    b = 2000 if n < 1 << 22 else 40          # (the oracle adds up all scores for each)
    assert np.array_equal(T.selector_draw(s, b, 3, 8).cpu().numpy(), oracle.batch_draw(score, b, seed=3, iteration=8))
    T.selector_free(s)
    s = T.selector_init(torch.zeros(n, dtype=torch.int32, device="cuda"))
    assert T.selector_draw(s, 5, 3, 8).tolist() == [-1] * 5
    T.selector_update(s, torch.tensor([n - 1], dtype=torch.int32, device="cuda"), torch.tensor([7], dtype=torch.int32, device="cuda"))
    assert T.selector_draw(s, 5, 3, 9).tolist() == [n - 1] * 5
    T.selector_free(s)
