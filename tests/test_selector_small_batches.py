"""Score updates around the line between one block and two launches, and draws from groups of every length."""
import numpy as np
import pytest
import torch

import oracle
import paper_2402_05396_amd as T

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("b", [5, 512, 1023, 1024, 1025, 6000])
@pytest.mark.parametrize("step", [1, 2048])
def test_repeated_and_colliding_edges(b, step):
    """Edges a multiple of 2048 apart share a slot of the block's hash table; each is named about four times,
    some entries are padding or out of range. The last value of an edge stays, the sums follow."""
    rng = np.random.default_rng(b + step)
    n = step * (b // 4) + 3
    score = rng.integers(1, 1 << 32, n, dtype=np.uint64).astype(np.uint32)
    s = T.selector_init(dev(score.view(np.int32)))
    idx = (rng.integers(0, b // 4, b) * step).astype(np.int32)
    idx[3::17], idx[5::19], idx[-1] = -1, n, n - 1
    val = rng.integers(0, 1 << 32, b, dtype=np.uint64).astype(np.uint32)
    oracle.score_update(score, idx, val)
    T.selector_update(s, dev(idx), dev(val.view(np.int32)))
    got, total = T.selector_scores(s)
    assert np.array_equal(got.cpu().numpy().view(np.uint32), score)
    assert total == int(score.astype(np.uint64).sum())
    assert np.array_equal(T.selector_draw(s, 3000, 5, 9).cpu().numpy(), oracle.batch_draw(score, 3000, seed=5, iteration=9))
    T.selector_free(s)


@pytest.mark.parametrize("n", [2, 255, 256, 257, 1023, 1280, 2048, 131073, 1024 * 128 * 2 + 1])
def test_draws_reach_every_row_of_a_group(n):
    """Equal scores: the draws spread over all rows (256 scores, 128 sums) of the groups and over their ends."""
    score = np.full(n, 0xFFFFFFFF, np.uint32)
    s = T.selector_init(dev(score.view(np.int32)))
    assert np.array_equal(T.selector_draw(s, 8000, 3, 1).cpu().numpy(), oracle.batch_draw(score, 8000, seed=3, iteration=1))
    T.selector_free(s)
