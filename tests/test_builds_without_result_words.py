"""Builds that find all page-locked result words taken, because more of them wait for their stream than there are: their results
come back over that stream, whatever the null stream is doing."""
import threading
import time

import numpy as np
import pytest
import torch

import oracle
import paper_2402_05396_amd as T

pytestmark = pytest.mark.gpu

BUILDS = 72          # 64 of them have words


def _inputs():
    """Input in no order whose buckets can be sorted, and input that has one bucket too large (all samples have one value)."""
    n = 20_000
    rng = np.random.default_rng(1)
    h = np.arange((n + 255) // 256, dtype=np.uint64) * 0x9E3779B1 % 2**32
    h = (h ^ (h >> np.uint64(15))) * 0x85EBCA77 % 2**32
    places = np.arange(len(h)) * 256 + ((h >> np.uint64(13)) % 256).astype(np.int64)
    places = places[places < n]
    src, ts = np.full(n, 50, np.int32), rng.integers(1000, 2000, n).astype(np.int64)
    src[places], ts[places] = 99, 5000
    return [(rng.integers(0, 100, n).astype(np.int32), rng.integers(0, 1 << 22, n).astype(np.int64)), (src, ts)]


def test_more_builds_at_a_time_than_result_words():
    dst, eid = np.arange(20_000, dtype=np.int32), np.arange(20_000, dtype=np.int32)
    inputs = [(src, ts, oracle.tcsr_build(src, dst, ts, eid, 100)) for src, ts in _inputs()]
    d_dst = torch.from_numpy(dst).cuda()
    columns = [(torch.from_numpy(src).cuda(), torch.from_numpy(ts).cuda()) for src, ts, _ in inputs]
    T.tcsr_free(T.tcsr_build(columns[0][0], d_dst, columns[0][1], None, 100))
    sizes = T.tcsr_build_bytes(20_000, 100)
    blocks = [[torch.empty(b, dtype=torch.uint8, device="cuda") for b in sizes] for _ in range(BUILDS)]
    begin, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    torch.cuda._sleep(1000)
    begin.record()
    torch.cuda._sleep(1_000_000)
    end.record()
    end.synchronize()
    second = int(1_000_000 * 1000 / max(begin.elapsed_time(end), 1e-3))          # in cycles
    streams = [torch.cuda.Stream() for _ in range(8)]
    torch.cuda.synchronize()

    torch.cuda._sleep(2 * second)                     # the null stream is busy
    ready = []
    for s in streams:                                 # one that does not share a queue with it
        with torch.cuda.stream(s):
            torch.cuda._sleep(1000)
            ready.append(s.record_event())
    time.sleep(0.1)
    free = [s for s, e in zip(streams, ready) if e.query()]
    assert free and not torch.cuda.default_stream().query()
    with torch.cuda.stream(free[0]):
        torch.cuda._sleep(second // 2)                # the builds wait behind this, each with its words
    graphs, errors, started, returned = [None] * BUILDS, [], [], []

    def build(i):
        started.append(i)
        try:
            graphs[i] = T.tcsr_build_in(columns[i % 2][0], d_dst, columns[i % 2][1], None, 100, *blocks[i], stream=free[0])
        except Exception as e:
            errors.append(repr(e))
        returned.append(i)

    threads = [threading.Thread(target=build, args=(i,)) for i in range(BUILDS)]
    for t in threads:
        t.start()
    time.sleep(0.1)
    waiting = len(started) - len(returned)
    for t in threads:
        t.join()
    still_busy = not torch.cuda.default_stream().query()
    torch.cuda.synchronize()
    assert waiting == BUILDS and not errors, (waiting, errors[:2])
    assert still_busy, "a build waited for the null stream"
    for i, g in enumerate(graphs):
        for got, want in zip(T.tcsr_view(g), inputs[i % 2][2]):
            assert np.array_equal(got.cpu().numpy(), want), i
        T.tcsr_free(g)
