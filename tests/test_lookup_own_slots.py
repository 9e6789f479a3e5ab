"""Lookups where the miss table has a slot per row (plain stores claim them) and, one row more, where it has not: the
table's last slots, tables that are no multiple of what a wave stages at a time, staging areas that are too small, and few
misses in large tables."""
import numpy as np
import pytest
import torch

import oracle
import paper_2402_05396_amd as T

pytestmark = pytest.mark.gpu


# the miss table has the power of two from 2 * staging_rows on, at least 64
@pytest.mark.parametrize("rows,staging", [(1, 1), (63, 32), (64, 32), (65, 32), (1000, 500), (1024, 512), (1025, 512), (4096, 1100), (4097, 1100)])
@pytest.mark.parametrize("dim", [3, 16, 413])
def test_every_row_can_be_missed_and_staged(rows, staging, dim):
    rng = np.random.default_rng(rows + dim)
    host = torch.from_numpy(rng.standard_normal((rows, dim)).astype(np.float32)).pin_memory()
    resident = np.sort(rng.permutation(rows)[:rows // 3]).astype(np.int32)
    c = T.cache_init(host, len(resident), torch.from_numpy(resident), staging_rows=staging)
    T.cache_count_accesses(c)
    counts = np.zeros(rows, np.uint32)
    few = np.array([rows - 1, 0, rows - 1, -1, rows], np.int32)
    every = rng.permutation(np.concatenate([np.arange(rows, dtype=np.int32)] * 3 + [np.full(4096, rows - 1, np.int32), few]))
    for ids_np in (few, every, few, every[::-1].copy()):   # each call finds the table as the one before left it
        known = np.where(ids_np >= rows, -1, ids_np)
        ids, hm = torch.from_numpy(ids_np).cuda(), torch.zeros(2, dtype=torch.int64, device="cuda")
        out = T.cache_lookup(c, ids, hit_miss=hm)
        assert out.cpu().numpy().tobytes() == oracle.gather(host.numpy(), known).tobytes()
        hits = int(np.isin(known[known >= 0], resident).sum())
        assert hm.tolist() == [hits, int((known >= 0).sum()) - hits]
        oracle.cache_count(known, rows, counts)
    assert np.array_equal(T.cache_access_counts(c).cpu().numpy().view(np.uint32), counts)
    T.cache_free(c)


@pytest.mark.parametrize("rows,dim", [(4095, 512), (4096, 512), (4097, 512), (36_864, 1024), (70_003, 300), (131_071, 260)])
@pytest.mark.parametrize("stage_blocks", [0, 3])
def test_waves_take_several_spans(rows, dim, stage_blocks):
    """Spans of 8 slots, of which a wave has several at once: one round of them, one more or less, several and a rest."""
    rng = np.random.default_rng(rows)
    host = torch.from_numpy(rng.standard_normal((rows, dim), dtype=np.float32)).pin_memory()
    table = torch.cat([host.cuda(), torch.zeros((1, dim), device="cuda")])
    resident = torch.from_numpy(np.sort(rng.permutation(rows)[:rows // 4]).astype(np.int32))
    few = torch.from_numpy(np.concatenate([[0, 7, 8, rows - 1, rows - 8, rows - 9], rng.integers(-1, rows, 500)]).astype(np.int32)).cuda()
    every = torch.from_numpy(rng.permutation(rows).astype(np.int32)).cuda()
    for staging in (rows, rows // 2 + 1, rows // 8):     # the last one: hashed slots, and too few rows
        c = T.cache_init(host, len(resident), resident, staging_rows=staging)
        T.cache_tune(c, stage_blocks=stage_blocks)
        for ids in (few, every, few):
            out = T.cache_lookup(c, ids)
            assert torch.equal(out, table[ids.long()]), (staging, len(ids))     # -1: the row of zeros at the end
        T.cache_free(c)


@pytest.mark.parametrize("rows,dim,staging", [(4096, 512, 2048), (36_864, 1024, 18_500), (70_003, 300, 40_000), (131_071, 260, 70_000), (8000, 8, 4000),
                                              (8200, 16, 8200)])
@pytest.mark.parametrize("stage_blocks", [0, 1, 3, 50])
def test_waves_begin_apart(rows, dim, staging, stage_blocks):
    """At most a quarter of the rows can be missed, by 8 192 requests and more: the waves go through the table from places of their own."""
    rng = np.random.default_rng(rows + 1)
    host = torch.from_numpy(rng.standard_normal((rows, dim), dtype=np.float32)).pin_memory()
    table = torch.cat([host.cuda(), torch.zeros((1, dim), device="cuda")])
    missing = np.unique(np.concatenate([[0, 7, 8, rows - 1, rows - 8, rows - 9], rng.permutation(rows)[:rows // 4 - 6]]))
    resident = torch.from_numpy(np.setdiff1d(np.arange(rows), missing).astype(np.int32))
    some, every = rng.choice(missing, 100), np.concatenate([missing, rng.integers(-1, rows, 9000)])
    c = T.cache_init(host, len(resident), resident, staging_rows=staging)
    T.cache_tune(c, stage_blocks=stage_blocks)
    for ids_np in (np.concatenate([some, np.full(8192 - 100, int(resident[0]))]), every, some, every[::-1].copy()):
        ids, hm = torch.from_numpy(ids_np.astype(np.int32)).cuda(), torch.zeros(2, dtype=torch.int64, device="cuda")
        out = T.cache_lookup(c, ids, hit_miss=hm)
        assert torch.equal(out, table[ids.long()]), len(ids)
        assert hm.tolist()[1] == int(np.isin(ids_np, missing).sum())
    T.cache_free(c)


def test_missing_rows_in_strides_are_every_waves():
    """938 missing rows whose ids are multiples of 64 take no longer than as many neighboring ones, as long as the spans that hold them go
    to different waves (163 us; 215 where they all went to every eighth)."""
    rows, dim, n = 60_000, 413, 400_000
    host = torch.randn((rows, dim), generator=torch.Generator().manual_seed(5)).pin_memory()
    pick = torch.randint(0, rows // 64 + 1, (n,), generator=torch.Generator(device="cuda").manual_seed(8), device="cuda", dtype=torch.int32)
    c, took = T.cache_init(host, 0, staging_rows=rows), {}
    for stride in (64, 1):
        ids, out = pick * stride, torch.empty((n, dim), device="cuda")
        T.cache_lookup(c, ids, out=out)
        assert torch.equal(out, host.cuda()[ids.long()])
        took[stride] = 1e9
        for _ in range(10):
            T.profile_begin()
            T.cache_lookup(c, ids, out=out)
            took[stride] = min(took[stride], T.profile_end()["cache_stage_and_gather_rows"][1])
    T.cache_free(c)
    assert took[64] < 1.3 * took[1], took


def test_few_misses_of_a_large_table_are_found_as_fast_with_a_slot_per_row():
    """500 requests of a million rows: looking through a slot per row may not take longer than through a hashed table of half
    as many slots by more than what the slots more are (24 and 22 us; 58 where waves looked at 8 slots at a time)."""
    rows, dim = 1_000_000, 172
    host = torch.zeros((rows, dim)).pin_memory()
    ids = torch.randint(0, rows, (500,), generator=torch.Generator(device="cuda").manual_seed(2), device="cuda", dtype=torch.int32)
    out, best = torch.empty((500, dim), device="cuda"), {}
    begin, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    for staging in (500_000, 250_000):
        c = T.cache_init(host, 500_000, None, seed=1, staging_rows=staging)
        times = []
        for _ in range(12):
            begin.record()
            for _ in range(20):
                T.cache_lookup(c, ids, out=out)
            end.record()
            end.synchronize()
            times.append(begin.elapsed_time(end))
        best[staging] = min(times)
        T.cache_free(c)
    assert best[500_000] < 1.35 * best[250_000], best
