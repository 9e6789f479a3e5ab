"""The inverse-timespan finder on lists with many entries 2^32 and more before the query: they all weigh 1, and are one run
that is not read."""
import numpy as np
import pytest
import torch

import oracle
import paper_2402_05396_amd as T

NOW = (1 << 52) + 12_345


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.gpu
@pytest.mark.parametrize("old", [1, 64, 255, 256, 257, 5000, 70_000])
@pytest.mark.parametrize("young,spread", [(0, 1), (1, 1 << 31), (70, 60_000), (600, 50_000), (600, 1 << 32), (30_000, 1 << 24), (30_000, 1 << 32)])
def test_old_entries_beside_every_kind_of_rest(old, young, spread):
    """`old` entries beyond 2^32 and `young` ones within `spread` before the query: no, few, near and far ones."""
    rng = np.random.default_rng(old + young)
    ts = np.sort(np.concatenate([NOW - rng.integers(1 << 32, 1 << 50, old), NOW - rng.integers(1, spread, young) if young else []])).astype(np.int64)
    n = ts.shape[0]
    ts[old - 1] = NOW - (1 << 32)
    src, dst, eid = np.zeros(n, np.int32), rng.integers(0, 9, n).astype(np.int32), np.arange(n, dtype=np.int32)
    g, g_ref = T.tcsr_build(_dev(src), _dev(dst), _dev(ts), _dev(eid), 9), oracle.tcsr_build(src, dst, ts, eid, 9, 8)
    times = np.array([NOW, NOW - 1, NOW + 1, ts[-1], ts[n // 2] + (1 << 32), NOW + (1 << 33)], np.int64)
    roots = np.zeros(times.shape[0], np.int32)
    for k in (1, 10, 64):
        want = oracle.sample_temporal(g_ref, roots, times, k, 1, T.INVERSE_TIMESPAN, 5)[0]
        got = T.sample_temporal(g, _dev(roots), _dev(times), k, 1, T.INVERSE_TIMESPAN, 5)[0]
        for f in ("nbr", "eid", "ts", "count"):
            assert np.array_equal(got[f].cpu().numpy(), want[f]), (k, f)


@pytest.mark.gpu
def test_old_entries_take_no_time():
    """50 young entries behind 4 000 and behind 4 000 000 old ones: one call takes about as long as the other (read, the
    longer list took thirty times as long)."""
    def microseconds(old):
        ts = torch.cat([torch.arange(old, device="cuda"), (1 << 40) + torch.arange(50, device="cuda")])
        node = torch.zeros(old + 50, dtype=torch.int32, device="cuda")
        g = T.tcsr_build(node, node, ts, None, 1)
        roots, times = torch.zeros(64, dtype=torch.int32, device="cuda"), torch.full((64,), (1 << 40) + 60, device="cuda")
        begin, end, best = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True), 1e9
        for _ in range(10):
            begin.record()
            for _ in range(10):
                T.sample_temporal(g, roots, times, 10, 1, T.INVERSE_TIMESPAN, 5)
            end.record()
            end.synchronize()
            best = min(best, begin.elapsed_time(end) * 100)
        return best

    few, many = microseconds(4000), microseconds(4_000_000)
    print(few, many)
    assert many < 4 * few
