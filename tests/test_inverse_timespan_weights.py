"""The inverse-timespan finder where its weights change form: spans on both sides of 2^16, 2^24, 2^31 and 2^32,
lists around a tile's and a row's ends, and the smallest and largest list it tiles."""
import os
import subprocess

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


def _ties(n, delta, ks):
    """One list of n entries, all of them delta before the queries."""
    ts = torch.zeros(n, dtype=torch.int64, device="cuda")
    src = torch.zeros(n, dtype=torch.int32, device="cuda")
    eid = torch.arange(n, dtype=torch.int32, device="cuda")
    g = T.tcsr_build(src, eid, ts, eid, 1)
    g_ref = oracle.tcsr_build(*(t.cpu().numpy() for t in (src, eid, ts, eid)), 1, THREADS)
    roots, times = np.zeros(5, np.int32), np.full(5, delta, np.int64)
    for k in ks:
        want = oracle.sample_temporal(g_ref, roots, times, k, 1, T.INVERSE_TIMESPAN, 3, threads=THREADS)[0]
        got = T.sample_temporal(g, torch.from_numpy(roots).cuda(), torch.from_numpy(times).cuda(), k, 1, T.INVERSE_TIMESPAN, 3)[0]
        for f in ("nbr", "eid", "ts", "count"):
            assert np.array_equal(got[f].cpu().numpy(), want[f]), (k, f)


@pytest.mark.gpu
@pytest.mark.parametrize("delta", [65_536, 65_537])
def test_tiles_of_ties_at_the_largest_weights(delta):
    """The shortest list whose tiles hold 1 024 rows of 64 entries (a block of one root has 1 024 tiles), all of them one
    timestamp: a full tile weighs 65 536 * 65 536 = 2^32 where delta is 65 536, and 65 536 * 65 535 one later."""
    _ties(1024 * 512 * 64 + 1, delta, (1, 10))


@pytest.mark.gpu
@pytest.mark.parametrize("delta", [1, 2, 63, 64, 65, 127, 128, 129])
@pytest.mark.parametrize("n", [8 * 64 - 1, 8 * 64, 8 * 64 + 1, 40 * 8 * 64 + 7])
def test_rows_of_ties_at_the_ends_of_32_bits(delta, n):
    """Groups of eight rows of 64 entries: a row weighs 64 * 2^26 = 2^32 at delta 64, 2^31 at the delta from which rows are
    summed in 32 bits (128), and a lane's eight rows 2^29 there."""
    _ties(n, delta, (1, 10, 64))


PROGRAM = r"""
#include "timespan_weight.h"
#include <math.h>
#include <random>
#include <stdio.h>
static int bad = 0;
static void check(uint64_t d) {
    if (d < 1 || d >> 32) return;
    const uint32_t delta = (uint32_t)d;
    const uint64_t want = ((uint64_t)1 << 32) / d;
    const float r = 1.0f / (float)delta, of[3] = {r, nextafterf(r, 2.0f), nextafterf(r, 0.0f)};
    for (int i = 0; i < 3; ++i) {
        bool ok = weight_by_reciprocal(delta, of[i]) == want;
        if (delta > kLastLargeDelta) ok = ok && quotient_by_reciprocal<false>(delta, of[i]) == want;
        if (delta > kLastLargeDelta && delta < 1u << 24) ok = ok && quotient_by_reciprocal<true>(delta, of[i]) == want;
        if (!ok && ++bad < 20) printf("delta %u, reciprocal %d\n", delta, i);
    }
}
int main() {
    for (uint64_t d = 1; d < (1u << 24) + 1000; ++d) check(d);
    for (uint64_t w = 1; w < 70000; ++w)
        for (int i = -2; i <= 2; ++i) check(((uint64_t)1 << 32) / w + i);
    for (int bit = 24; bit <= 32; ++bit)
        for (int i = -3000; i <= 3000; ++i) check(((uint64_t)1 << bit) + i);
    std::mt19937_64 rng(1);
    for (int i = 0; i < 3000000; ++i) check(rng() >> (32 + rng() % 9));
    return bad != 0;
}
"""


def test_the_weight_of_a_delta_is_exact_whatever_the_reciprocals_last_bit(tmp_path):
    """The kernel's own functions (csrc/timespan_weight.h) in a CPU program: every delta below 2^24, and those above it at which
    the quotient changes."""
    csrc = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2402_05396_amd", "csrc")
    (tmp_path / "w.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O2", "-w", "-D__HIP_PLATFORM_AMD__=1", "-I", csrc, "-isystem", "/opt/rocm/include", "-o", str(tmp_path / "w"),
                    str(tmp_path / "w.cpp")], check=True)
    r = subprocess.run([str(tmp_path / "w")], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
