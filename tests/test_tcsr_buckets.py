"""Builds from input in no order that is cut into buckets: sizes around one bucket, a tile and the largest input, keys that all
agree, buckets of one node's entries, long spans, and input whose buckets cannot be sorted, which the digit passes take over."""
import numpy as np
import pytest
import torch

import oracle
import paper_2402_05396_amd as T

pytestmark = pytest.mark.gpu


def _check(src, ts, num_nodes, eid=None):
    n = len(src)
    dst = ((np.arange(n, dtype=np.int64) * 7919) % 2_000_000_011).astype(np.int32)
    d = lambda a: None if a is None else torch.from_numpy(np.ascontiguousarray(a)).cuda()
    ref = oracle.tcsr_build(src, dst, ts, np.arange(n, dtype=np.int32) if eid is None else eid, num_nodes)   # indptr, nbr, ts, eid
    g = T.tcsr_build(d(src), d(dst), d(ts), d(eid), num_nodes)
    indptr, nbr, times, eids = T.tcsr_view(g)
    for got, want in zip((indptr, nbr, times, eids), ref):
        assert np.array_equal(got.cpu().numpy(), want)
    # the search index: every list cut at a time in the middle of it
    roots = np.unique(src)[:500].astype(np.int32)
    at = np.full(len(roots), int(np.median(ts)), np.int64)
    out = T.sample_temporal(g, d(roots), d(at), 7, 1, T.RECENT, 0)[0]
    want = oracle.sample_temporal(ref, roots, at, 7, 1, T.RECENT, 0)[0]
    assert np.array_equal(out["eid"].cpu().numpy(), want["eid"]) and np.array_equal(out["count"].cpu().numpy(), want["count"])


@pytest.mark.parametrize("n", [2, 63, 64, 65, 2047, 2048, 2049, 4095, 4096, 4097, 6145, 20_000, 100_001, 1_048_577, 1_572_864, 1_572_865])
@pytest.mark.parametrize("num_nodes,span", [(1, 1 << 20), (1000, 50), (11_000, 1 << 22)])
def test_sizes(n, num_nodes, span):
    rng = np.random.default_rng(n + num_nodes)
    src = np.minimum(rng.zipf(1.2, n) - 1, num_nodes - 1).astype(np.int32)
    ts = rng.integers(-span // 2, span // 2, n).astype(np.int64)
    ts[:2] = span, 0                                     # not in order, whatever else there is
    _check(src, ts, num_nodes, rng.permutation(n).astype(np.int32) if n % 2 else None)


@pytest.mark.parametrize("n", [524_288, 524_289])
@pytest.mark.parametrize("num_nodes", [1 << 12, 1 << 13])
def test_few_key_bits(n, num_nodes):
    """27 and 28 bits of key on both sides of the size from which the former go through the digit passes."""
    rng = np.random.default_rng(n + num_nodes)
    ts = rng.integers(0, 1 << 15, n).astype(np.int64)
    ts[:2] = (1 << 15) - 1, 0
    _check(rng.integers(0, num_nodes, n).astype(np.int32), ts, num_nodes)


@pytest.mark.parametrize("kind", ["ties", "two_times", "one_node_late", "blocks", "reversed", "nearly"])
def test_orders(kind):
    rng = np.random.default_rng(5)
    n, num_nodes = 300_000, 5000
    src = rng.integers(0, num_nodes, n).astype(np.int32)
    ts = rng.integers(0, 1 << 30, n).astype(np.int64)
    if kind == "ties":
        src[:], ts[:] = 17, 5
        ts[0] = 6                                        # all other keys agree: the position cuts them
    elif kind == "two_times":
        ts = rng.integers(0, 2, n).astype(np.int64) << 40
    elif kind == "one_node_late":
        src[n // 2:] = 4999
    elif kind == "blocks":
        ts = np.concatenate([np.sort(x) for x in np.split(ts, 100)])
    elif kind == "reversed":
        ts = np.sort(ts)[::-1].copy()
    else:
        ts = np.sort(ts)
        ts[n // 3], ts[n // 3 + 1] = ts[n // 3 + 1] + 1, ts[n // 3]
    _check(src, ts, num_nodes)


@pytest.mark.parametrize("n", [300, 4097, 70_000])
@pytest.mark.parametrize("node_bits,span_bits", [(20, 31), (20, 32), (1, 50), (1, 51), (0, 51), (24, 27), (14, 45), (3, 64)])
def test_long_keys(n, node_bits, span_bits):
    """Keys of up to 51 bits go into buckets, longer ones through the digit passes."""
    rng = np.random.default_rng(n + node_bits)
    src = rng.integers(0, 1 << node_bits, n).astype(np.int32)
    low, high = (-(1 << 63), (1 << 63) - 1) if span_bits == 64 else (0, 1 << span_bits)
    ts = rng.integers(low, high, n, dtype=np.int64)
    ts[0], ts[1] = high - 1, low
    src[0] = (1 << node_bits) - 1
    _check(src, ts, 1 << node_bits)


def test_a_bucket_too_large():
    """The samples are taken at fixed places. With one value at all of them every other entry is between two of them."""
    n, num_nodes = 400_000, 100
    h = np.arange((n + 255) // 256, dtype=np.uint64) * 0x9E3779B1 % 2**32
    h = (h ^ (h >> np.uint64(15))) * 0x85EBCA77 % 2**32
    places = np.arange(len(h)) * 256 + ((h >> np.uint64(13)) % 256).astype(np.int64)
    rng = np.random.default_rng(3)
    src, ts = np.full(n, 50, np.int32), rng.integers(1000, 2000, n).astype(np.int64)
    src[places[places < n]] = 99
    ts[places[places < n]] = 5000
    _check(src, ts, num_nodes)
