"""The finder at the edges of its rules: the most-recent hop size that changes kernels, lists that end with the
arrays its search reads in whole groups, and weights on both sides of the 32-bit draws."""
import numpy as np
import pytest
import torch

import oracle
import paper_2402_05396_amd as T

pytestmark = pytest.mark.gpu
THREADS = min(16, oracle.max_threads())


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def both(src, dst, ts, nodes):
    eid = np.arange(src.shape[0], dtype=np.int32)
    return T.tcsr_build(dev(src), dev(dst), dev(ts), dev(eid), nodes), oracle.tcsr_build(src, dst, ts, eid, nodes, THREADS)


def compare(g, g_ref, roots, times, k, hops, policy, m=0, weight=None):
    known = np.where(roots < g.num_nodes, roots, -1)     # the oracle takes no id beyond the graph's
    want = oracle.sample_temporal(g_ref, known, times, k, hops, policy, 11, m, weight, THREADS)
    got = T.sample_temporal(g, dev(roots), dev(times), k, hops, policy, 11, m, None if weight is None else dev(weight.view(np.int32)))
    for h in range(hops):
        for f in ("nbr", "eid", "ts", "count"):
            assert np.array_equal(got[h][f].cpu().numpy(), want[h][f]), (h, f)


@pytest.mark.parametrize("entries", [0, 1, 15, 16, 17, 255, 256, 257, 4096, 65536, 70_001])
@pytest.mark.parametrize("n,k", [(16_383, 10), (16_384, 1), (16_385, 3), (16_384 + 17, 10), (20_000, 25), (17_001, 64),
                                 (16_384, 33), (20_480, 32), (24_575, 10), (24_577, 13), (32_768 + 5, 10), (32_769, 28), (40_960 + 17, 1), (40_961, 4), (41_001, 25), (40_960 + 1, 50), (65_535, 16), (65_536, 31), (65_537, 16)])
def test_recent_around_the_large_hop(entries, n, k):
    rng = np.random.default_rng(entries + n)
    nodes = 3 if entries < 5000 else 40
    src = np.sort(rng.integers(0, nodes, entries)).astype(np.int32)
    src[entries // 2:] = nodes - 1                       # the last node's list runs to the end of the arrays
    dst = rng.integers(0, nodes, entries).astype(np.int32)
    ts = np.sort(rng.integers(-50, 2000, entries)).astype(np.int64)
    g, g_ref = both(src, dst, ts, nodes)
    roots = rng.integers(-1, nodes + 1, n).astype(np.int32)
    times = rng.integers(-60, 2010, n).astype(np.int64)
    times[:5] = [-(1 << 63), (1 << 63) - 1, 0, 2000, -50]
    compare(g, g_ref, roots, times, k, 1, T.RECENT)


def test_recent_second_hop_is_the_large_one():
    rng = np.random.default_rng(5)
    src, dst = rng.integers(0, 500, (2, 40_000)).astype(np.int32)
    ts = np.sort(rng.integers(0, 9000, 40_000)).astype(np.int64)
    g, g_ref = both(src, dst, ts, 500)
    for n in (1700, 3300):
        compare(g, g_ref, rng.integers(0, 500, n).astype(np.int32), rng.integers(0, 9001, n).astype(np.int64), 10, 2, T.RECENT)


@pytest.mark.parametrize("k,m", [(1, 2), (5, 16), (10, 25), (31, 32), (10, 64), (63, 64)])
@pytest.mark.parametrize("top", [1, 65536, (1 << 26) - 1, 1 << 26, (1 << 32) - 1])
def test_weights_on_both_sides_of_the_32_bit_draws(k, m, top):
    rng = np.random.default_rng(k * m)
    src = rng.integers(0, 30, 6000).astype(np.int32)
    ts = np.sort(rng.integers(0, 5000, 6000)).astype(np.int64)
    g, g_ref = both(src, rng.integers(0, 30, 6000).astype(np.int32), ts, 30)
    weight = rng.integers(max(1, top - 1000), top + 1, 6000).astype(np.uint32)
    weight[::7] = 1
    roots, times = rng.integers(-1, 30, 301).astype(np.int32), rng.integers(0, 5001, 301).astype(np.int64)
    compare(g, g_ref, roots, times, k, 1, T.WEIGHTED, m, weight)
    # per-slot weights (at least 1) through the window's own selection
    count = rng.integers(0, m + 1, 301).astype(np.int32)
    w = rng.integers(max(1, top - 1000), top + 1, (301, m)).astype(np.uint32)
    w[::5] = 1
    w[::5, m // 2] = top
    want = oracle.select_weighted(w, count, k, 3, 1)
    got = T.select_weighted(dev(w.view(np.int32)), dev(count), k, 3, 1)
    for a, b in zip(got[:2], want[:2]):
        assert np.array_equal(a.cpu().numpy(), b)


@pytest.mark.parametrize("dtype,dim,pad,n,k", [(np.float32, 300, 0, 37, 5), (np.float16, 413, 0, 29, 6), (np.float16, 172, 20, 40, 4), (np.float32, 1030, 0, 1, 3)])
def test_rows_of_three_hops_in_one_gather_launch(dtype, dim, pad, n, k):
    """Rows too long for the hop kernels: one launch gathers all hops' rows where every buffer is 16-byte aligned, one per
    hop where one is not; the hops' last blocks are partial."""
    rng = np.random.default_rng(dim)
    src, dst = rng.integers(0, 60, (2, 900)).astype(np.int32)
    ts = np.sort(rng.integers(0, 700, 900)).astype(np.int64)
    g, g_ref = both(src, dst, ts, 60)
    full = rng.integers(-2 ** 15, 2 ** 15, (800, (dim + pad) * np.dtype(dtype).itemsize // 2)).astype(np.int16).view(dtype)   # ids from 800 on: zero rows
    table, table_np = dev(full)[:, :dim], full[:, :dim]
    roots, times = rng.integers(-1, 60, n).astype(np.int32), rng.integers(300, 701, n).astype(np.int64)
    want = oracle.sample_temporal(g_ref, roots, times, k, 3, T.RECENT, 1, 0, None, THREADS)
    out, rows = T.sample_temporal_rows(g, dev(roots), dev(times), k, 3, T.RECENT, 1, table)
    odd = [torch.empty(w["eid"].size * dim + 8, dtype=table.dtype, device="cuda")[(2 if h == 1 else 0):][:w["eid"].size * dim].view(-1, dim)
           for h, w in enumerate(want)]
    _, rows2 = T.sample_temporal_rows(g, dev(roots), dev(times), k, 3, T.RECENT, 1, table, out=T.sample_outputs(n, k, 3, "cuda"), rows_out=odd)
    for h in range(3):
        assert np.array_equal(out[h]["eid"].cpu().numpy(), want[h]["eid"])
        ids = want[h]["eid"].ravel()
        bytes_ = oracle.gather(np.ascontiguousarray(table_np), np.where(ids >= 800, -1, ids)).tobytes()
        assert rows[h].cpu().numpy().tobytes() == bytes_ and rows2[h].cpu().numpy().tobytes() == bytes_, h
