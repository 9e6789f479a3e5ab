"""Score updates of medium batches: blocks that share the batch by the edges' hash."""
import numpy as np
import pytest
import torch

import oracle
import paper_2402_05396_amd as T

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _hash(e):
    e = e.astype(np.uint64)
    m = np.uint64(0xffffffff)
    e ^= e >> np.uint64(16)
    e = e * np.uint64(0x9E3779B1) & m
    e ^= e >> np.uint64(15)
    e = e * np.uint64(0xBB67AE85) & m
    return e ^ (e >> np.uint64(16))


def _check(n, score, idx, val):
    s = T.selector_init(dev(score.view(np.int32)))
    for _ in range(2):      # the second time nothing changes
        oracle.score_update(score, idx, val)
        T.selector_update(s, dev(idx), dev(val.view(np.int32)))
        got, total = T.selector_scores(s)
        assert np.array_equal(got.cpu().numpy().view(np.uint32), score)
        assert total == int(score.astype(np.uint64).sum())
    assert np.array_equal(T.selector_draw(s, 500, 5, 9).cpu().numpy(), oracle.batch_draw(score, 500, seed=5, iteration=9))
    T.selector_free(s)


@pytest.mark.parametrize("b", [768, 769, 1024, 1025, 2047, 2048, 2049, 4095, 4096, 4097])
@pytest.mark.parametrize("n,distinct", [(3, 3), (50_000, 700), (3_000_000, 3_000_000)])
def test_the_last_value_of_an_edge_stays(b, n, distinct):
    rng = np.random.default_rng(b + n)
    score = rng.integers(1, 1 << 32, n, dtype=np.uint64).astype(np.uint32)
    idx = rng.integers(0, distinct, b).astype(np.int32)
    idx[3::17], idx[5::19], idx[7::23], idx[-1] = -1, n, np.iinfo(np.int32).min, n - 1
    _check(n, score, idx, rng.integers(0, 1 << 32, b, dtype=np.uint64).astype(np.uint32))


@pytest.mark.parametrize("b,bits", [(2048, 3), (4096, 4)])
def test_a_batch_that_is_one_blocks(b, bits):
    """All edges of one class, all of them different: the block's table takes the whole batch."""
    n = 200_000
    edges = np.arange(n)
    mine = edges[(_hash(edges) >> np.uint64(32 - bits)) == 5][:b].astype(np.int32)
    assert mine.shape[0] == b
    rng = np.random.default_rng(b)
    _check(n, np.full(n, 7, np.uint32), rng.permutation(mine), rng.integers(0, 1 << 32, b, dtype=np.uint64).astype(np.uint32))


@pytest.mark.parametrize("n", [64 << 20, (64 << 20) + 1])
def test_as_many_level_two_sums_as_a_block_holds(n):
    rng = np.random.default_rng(1)
    idx = rng.integers(0, n, 1500).astype(np.int32)
    idx[:64] = np.arange(64) << 20
    idx[-1] = n - 1
    _check(n, np.ones(n, np.uint32), idx, rng.integers(0, 1 << 32, 1500, dtype=np.uint64).astype(np.uint32))
