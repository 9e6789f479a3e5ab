"""Lookups where the miss table has a slot per row (plain stores claim them) and, one row more, where it has not: the
table's last slots, tables that are no multiple of what a wave stages at a time, and staging areas that are too small."""
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
