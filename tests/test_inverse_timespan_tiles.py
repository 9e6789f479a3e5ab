"""The inverse-timespan finder at the most tiles that a list is cut into, which depends on the roots of a block."""
import numpy as np
import pytest
import torch

import oracle
import paper_2402_05396_amd as T


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.gpu
@pytest.mark.parametrize("more", [-1, 0, 1])
@pytest.mark.parametrize("roots,full", [(5, 1024), (3000, 512), (4100, 256)])
def test_as_many_tiles_as_there_are(roots, full, more):
    """64 draws make tiles of sqrt(rows / 64) rows: full ** 2 / 64 rows of 64 entries are `full` tiles, one entry more is one too
    many. Few of the roots look at the list, which the first ticks hold all of (no part of it is summed by weights)."""
    n = full * full + more
    rng = np.random.default_rng(n)
    ts = np.sort(rng.integers(0, 30_000, n)).astype(np.int64)
    src, eid = np.zeros(n, np.int32), np.arange(n, dtype=np.int32)
    g, g_ref = T.tcsr_build(_dev(src), _dev(src), _dev(ts), _dev(eid), 2), oracle.tcsr_build(src, src, ts, eid, 2, 8)
    q, t = np.ones(roots, np.int32), np.full(roots, 30_000, np.int64)
    q[[0, 3, roots - 1]] = 0
    want = oracle.sample_temporal(g_ref, q, t, 64, 1, T.INVERSE_TIMESPAN, 5, threads=8)[0]
    got = T.sample_temporal(g, _dev(q), _dev(t), 64, 1, T.INVERSE_TIMESPAN, 5)[0]
    for f in ("nbr", "eid", "ts", "count"):
        assert np.array_equal(got[f].cpu().numpy(), want[f]), f


@pytest.mark.gpu
def test_draws_of_a_long_list_read_little_of_it():
    """200 roots over lists of a million entries: 64 draws take less than three times as long as one (1.6 times; six times with
    tiles of 128 rows)."""
    n = 4_000_000
    src = torch.arange(n, device="cuda", dtype=torch.int32) % 4
    ts = torch.arange(n, device="cuda") * 30_000 // n
    g = T.tcsr_build(src, src, ts, None, 4)
    roots, times = torch.arange(200, device="cuda", dtype=torch.int32) % 4, torch.full((200,), 29_000, device="cuda")

    def milliseconds(k):
        begin, end, best = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True), 1e9
        for _ in range(10):
            begin.record()
            T.sample_temporal(g, roots, times, k, 1, T.INVERSE_TIMESPAN, 5)
            end.record()
            end.synchronize()
            best = min(best, begin.elapsed_time(end))
        return best

    one, all_lanes = milliseconds(1), milliseconds(64)
    print(one, all_lanes)
    assert all_lanes < 3 * one
