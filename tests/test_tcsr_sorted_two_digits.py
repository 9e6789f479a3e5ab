"""tcsr_build on time-sorted input whose node ids take two digits: narrow records between the passes, list starts from the
scanned histogram."""
import numpy as np
import pytest
import torch

import paper_2402_05396_amd as T

# entries around the 2 048-item tiles of small builds, and around the 4 096-item ones from 2^21 entries on
SIZES = [1, 2047, 2048, 2049, 6144, 100_003, (1 << 21) + 1, (1 << 21) + 4096 * 3]


def _check(src, ts, nodes, eid=None):
    n = src.shape[0]
    dst = np.arange(n, dtype=np.int32)[::-1].copy() - 7       # a neighbor may be any number
    dev = lambda a: None if a is None else torch.from_numpy(a).cuda()
    g = T.tcsr_build(dev(src), dev(dst), dev(ts), dev(eid), nodes)
    indptr, nbr, t, e = (x.cpu().numpy() for x in T.tcsr_view(g))
    order = np.argsort(src, kind="stable")
    assert np.array_equal(indptr, np.searchsorted(src[order], np.arange(nodes + 1)))
    assert np.array_equal(nbr, dst[order]) and np.array_equal(t, ts[order])
    assert np.array_equal(e, (np.arange(n, dtype=np.int32) if eid is None else eid)[order])
    # the search index (made from the same pass): the most recent entry of every node that has one, just after the last time
    roots = np.arange(min(nodes, 5000), dtype=np.int32)
    if ts[-1] < np.iinfo(np.int64).max:
        got = T.sample_temporal(g, dev(roots), dev(np.full(roots.shape[0], ts[-1] + 1, np.int64)), 1, 1, T.RECENT, 0)[0]
        last = indptr[roots + 1] - 1
        want = np.where(last >= indptr[roots], e[np.maximum(last, 0)], -1)
        assert np.array_equal(got["eid"].cpu().numpy()[:, 0], want)


@pytest.mark.gpu
@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("nodes", [512, 513, 1024, 17_000, 65_536, 65_537, 262_144, 262_145])
def test_node_counts_on_both_sides_of_two_digits(n, nodes):
    rng = np.random.default_rng(n + nodes)
    src = np.minimum(rng.zipf(1.3, n) - 1, nodes - 1).astype(np.int32) if n % 2 else rng.integers(0, nodes, n).astype(np.int32)
    _check(src, np.sort(rng.integers(0, 1 << 31, n)).astype(np.int64), nodes, rng.integers(0, n + 5, n).astype(np.int32))


@pytest.mark.gpu
@pytest.mark.parametrize("first", [0, -(1 << 63), -5, (1 << 63) - (1 << 33), (1 << 32) - 3])
@pytest.mark.parametrize("span", [0, (1 << 32) - 1, 1 << 32, (1 << 32) + 1])
def test_spans_around_32_bits(first, span):
    n, rng = 5000, np.random.default_rng(span % 97)
    ts = (np.sort(rng.integers(0, span + 1, n)) + 0).astype(np.int64)
    ts[0], ts[-1] = 0, span
    _check(rng.integers(0, 3000, n).astype(np.int32), ts + np.int64(first), 3000)


@pytest.mark.gpu
@pytest.mark.parametrize("node", [0, 31, 32, 1023, 511])
def test_one_node_has_everything(node):
    n = 4096 * 2
    _check(np.full(n, node, np.int32), np.arange(n, dtype=np.int64), 1024)


@pytest.mark.gpu
@pytest.mark.parametrize("at", [0, 2046, 2047, 4095, 9_998])
def test_one_entry_out_of_time_order(at):
    """The entry after `at` is earlier: sorted by time as well, whatever place of a tile or a wave it has."""
    n, rng = 10_000, np.random.default_rng(at)
    ts = np.arange(10, n + 10, dtype=np.int64) * 3
    ts[at + 1] = ts[at] - 1
    src = np.full(n, 700, np.int32)
    g = T.tcsr_build(*(torch.from_numpy(x).cuda() for x in (src, src, ts, np.arange(n, dtype=np.int32))), 1024)
    order = np.argsort(ts, kind="stable")
    assert np.array_equal(T.tcsr_view(g)[2].cpu().numpy(), ts[order]) and np.array_equal(T.tcsr_view(g)[3].cpu().numpy(), order)


@pytest.mark.gpu
@pytest.mark.parametrize("nodes,passes", [(512, 1), (600, 2), (1025, 2), (17_000, 2), (131_072, 2), (131_073, 2), (262_144, 2), (262_145, 3)])
def test_a_long_span_counts_its_first_digit_in_the_inspection(nodes, passes):
    """In time order, but over 2^32 ticks and more: one histogram launch per digit after the first, whatever the digits' widths."""
    n, rng = 9000, np.random.default_rng(nodes)
    src = rng.integers(0, nodes, n).astype(np.int32)
    ts = np.sort(rng.integers(0, 1 << 45, n)).astype(np.int64)
    dev = [torch.from_numpy(x).cuda() for x in (src, src, ts)]
    T.profile_begin()
    T.tcsr_build(*dev, None, nodes)
    kernels = T.profile_end()
    assert kernels["tcsr_radix_scatter"][0] == passes and kernels.get("tcsr_radix_hist", (0, 0))[0] == passes - 1
    _check(src, ts, nodes)
