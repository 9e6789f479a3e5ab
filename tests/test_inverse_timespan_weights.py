"""The inverse-timespan finder where its weights change form: spans on both sides of 2^16, 2^24, 2^31 and 2^32,
lists around a tile's and a row's ends, and the smallest and largest list it tiles."""
import numpy as np
import pytest
import torch

import oracle
import paper_2402_05396_amd as T

THREADS = min(16, oracle.max_threads())


@pytest.mark.gpu
@pytest.mark.parametrize("n", [11, 63, 64, 65, 129, 4097, 40_000, 600_000])
@pytest.mark.parametrize("near,far", [(1, 300), (65_530, 65_545), (1, 1 << 24), (1 << 23, (1 << 24) - 1), (1, (1 << 24) + 1), (70_000, 1 << 31),
                                      ((1 << 31) - 40, (1 << 31) + 40), ((1 << 32) - 500, (1 << 32) + 500), (1, 1 << 40), (1 << 32, 1 << 33)])
def test_picks_equal_the_oracle(n, near, far):
    """One node's list of n entries, all of them between `near` and `far` before the latest query."""
    rng = np.random.default_rng(n + far % 1000)
    now = -(1 << 62) + 5 * far                       # low words that wrap, and a time below zero
    ts = np.sort(now - rng.integers(near, far + 1, n)).astype(np.int64)
    ts[0], ts[-1] = now - far, now - near
    src, dst, eid = np.zeros(n, np.int32), rng.integers(0, 50, n).astype(np.int32), np.arange(n, dtype=np.int32)
    dev = lambda a: torch.from_numpy(a).cuda()
    g = T.tcsr_build(dev(src), dev(dst), dev(ts), dev(eid), 50)
    g_ref = oracle.tcsr_build(src, dst, ts, eid, 50, 4)
    times = np.concatenate([[now, now + 1, ts[n // 2], ts[-1], ts[min(10, n - 1)] + 1], rng.integers(ts[0], now + 3, 27)]).astype(np.int64)
    roots = np.zeros(times.shape[0], np.int32)
    for k in (1, 10, 64):
        want = oracle.sample_temporal(g_ref, roots, times, k, 1, T.INVERSE_TIMESPAN, 7)[0]
        got = T.sample_temporal(g, dev(roots), dev(times), k, 1, T.INVERSE_TIMESPAN, 7)[0]
        for f in ("nbr", "eid", "ts", "count"):
            assert np.array_equal(got[f].cpu().numpy(), want[f]), (k, f)


@pytest.mark.gpu
@pytest.mark.parametrize("delta", [65_536, 65_537])
def test_tiles_of_ties_at_the_largest_weights(delta):
    """The shortest list whose tiles hold 1 024 rows of 64 entries, all of them one timestamp: a full tile weighs
    65 536 * 65 536 = 2^32 where delta is 65 536, and 65 536 * 65 535 one later."""
    n = 1023 * 512 * 64 + 1
    ts = torch.zeros(n, dtype=torch.int64, device="cuda")
    src = torch.zeros(n, dtype=torch.int32, device="cuda")
    eid = torch.arange(n, dtype=torch.int32, device="cuda")
    g = T.tcsr_build(src, eid, ts, eid, 1)
    g_ref = oracle.tcsr_build(*(t.cpu().numpy() for t in (src, eid, ts, eid)), 1, THREADS)
    roots, times = np.zeros(5, np.int32), np.full(5, delta, np.int64)
    for k in (1, 10):
        want = oracle.sample_temporal(g_ref, roots, times, k, 1, T.INVERSE_TIMESPAN, 3, threads=THREADS)[0]
        got = T.sample_temporal(g, torch.from_numpy(roots).cuda(), torch.from_numpy(times).cuda(), k, 1, T.INVERSE_TIMESPAN, 3)[0]
        for f in ("nbr", "eid", "ts", "count"):
            assert np.array_equal(got[f].cpu().numpy(), want[f]), (k, f)


def _quotient(delta, near):
    """The device's arithmetic for delta > 65536 in numpy: float32 products, the reciprocal off by up to one unit in the
    last place either way, then the remainder's correction."""
    d = delta.astype(np.float32)
    r = np.float32(1) / d
    out = []
    for off in (np.float32(0), np.float32(np.inf), np.float32(-np.inf)):
        rr = r if off == 0 else np.nextafter(r, off)
        q = (np.float32(4294967296.0 * (1 - 2.0 ** -21)) * rr).astype(np.float32).astype(np.uint64)
        rest = (2 ** 32 - q * delta) % 2 ** 32
        w = q + (rest >= delta)
        out.append(w if near else np.maximum(w, 1))
    return out


def test_the_quotient_is_exact_whatever_the_reciprocals_last_bit():
    rng = np.random.default_rng(1)
    q = rng.integers(1, 65536, 200_000).astype(np.uint64)
    edges = np.concatenate([2 ** 32 // q, 2 ** 32 // q + 1, rng.integers(65536, 2 ** 32, 400_000).astype(np.uint64),
                            np.arange(65536, 66000), np.arange(2 ** 24 - 300, 2 ** 24 + 300), np.arange(2 ** 31 - 300, 2 ** 31 + 300),
                            np.arange(2 ** 32 - 300, 2 ** 32)]).astype(np.uint64)
    edges = edges[(edges >= 65536) & (edges < 2 ** 32)]
    for got in _quotient(edges, False):
        assert np.array_equal(got, np.maximum(2 ** 32 // edges, 1))
    edges = edges[edges < 2 ** 24]
    for got in _quotient(edges, True):
        assert np.array_equal(got, 2 ** 32 // edges)
