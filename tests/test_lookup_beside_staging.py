"""The one-call lookup, which writes what needs only resident rows while the missing ones are staged: rows and
requests around the edges of its lines, pieces, tiles and staging groups, next to the two separate calls."""
import numpy as np
import pytest
import torch

import oracle
import paper_2402_05396_amd as T

pytestmark = pytest.mark.gpu


def _requests(rng, rows, n, kind):
    if kind == "zipf":
        ids = np.minimum(rng.zipf(1.2, n) - 1, rows - 1)
    elif kind == "alternate":                     # a resident (even) and a missing (odd) row in turn
        ids = 2 * rng.integers(0, rows // 2, n) + np.arange(n) % 2
    else:                                         # runs of missing rows between runs of resident ones
        ids = 2 * rng.integers(0, rows // 2, n) + (np.arange(n) // 37) % 2
    ids = ids.astype(np.int32)
    ids[3::59], ids[11::83] = -1, rows            # zero rows among them
    ids[-1] = rows - 1
    return ids


@pytest.mark.parametrize("dim,n", [(1, 70_001), (3, 5000), (4, 4097), (5, 1025), (16, 9001), (33, 2047),   # flat gather, short rows
                                   (127, 4096), (128, 4095),                                               # its last sizes
                                   (128, 4096), (129, 4096), (155, 5003), (413, 4999), (1025, 4096), (4096, 4100)])
@pytest.mark.parametrize("kind", ["zipf", "alternate", "runs"])
def test_lookup_equals_the_oracle(dim, n, kind):
    rng = np.random.default_rng(dim * 13 + n)
    rows = 2000
    host = torch.from_numpy(rng.standard_normal((rows, dim + 1)).astype(np.float32)).pin_memory()[:, :dim]
    residents = torch.arange(0, rows, 2, dtype=torch.int32)
    ids_np = _requests(rng, rows, n, kind)
    ids = torch.from_numpy(ids_np).cuda()
    want = oracle.gather(np.ascontiguousarray(host.numpy()), np.where(ids_np >= rows, -1, ids_np)).tobytes()
    for staging, stage_blocks in ((1000, 0), (1000, 1), (300, 32), (7, 5), (0, 3)):   # ample, too small, none
        c = T.cache_init(host, 1000, residents, staging_rows=staging)
        T.cache_tune(c, stage_blocks=stage_blocks)
        T.cache_count_accesses(c)
        for _ in range(2):                        # the second call finds what the first one left behind
            hm = torch.zeros(2, dtype=torch.int64, device="cuda")
            buf = torch.full((n * dim + 40,), 7.0, dtype=torch.float32, device="cuda")
            out = buf[:n * dim].view(n, dim)
            T.cache_lookup(c, ids, out=out, hit_miss=hm)
            assert out.cpu().numpy().tobytes() == want, (staging, "one call")
            assert bool((buf[n * dim:] == 7.0).all())
            valid = (ids_np >= 0) & (ids_np < rows)
            assert tuple(hm.tolist()) == (int((valid & (ids_np % 2 == 0)).sum()), int((valid & (ids_np % 2 == 1)).sum()))
            out.fill_(3.0)
            T.cache_gather(c, ids, out=out)       # accepted: the lookup of these ids was their prefetch as well
            assert out.cpu().numpy().tobytes() == want, (staging, "gather after the lookup")
            out.fill_(3.0)
            T.cache_prefetch(c, ids, hit_miss=hm)
            T.cache_gather(c, ids, out=out)
            assert out.cpu().numpy().tobytes() == want, (staging, "two calls")
            misaligned = torch.full((n * dim + 8,), 7.0, dtype=torch.float32, device="cuda")[1:1 + n * dim].view(n, dim)
            T.cache_lookup(c, ids, out=misaligned)
            assert misaligned.cpu().numpy().tobytes() == want, (staging, "4-byte aligned output")
        counts = T.cache_access_counts(c).cpu().numpy()
        Q = np.zeros(rows, np.uint32)
        for _ in range(6):                        # two lookups and one prefetch per round count
            oracle.cache_count(np.where(ids_np >= rows, -1, ids_np), rows, Q)
        assert np.array_equal(counts.view(np.uint32), Q)
        T.cache_free(c)


@pytest.mark.parametrize("dim,n", [(128, 4097), (413, 5001), (413, 70_003), (155, 330_001), (16, 9001)])
@pytest.mark.parametrize("resident", [0, 150, 900, 1990, 2000])
def test_lookup_whatever_the_share_of_misses(dim, n, resident):
    """From none to all of the requests missing, which decides how the second launch writes them: small launches, and
    ones whose workgroups take several units."""
    rng = np.random.default_rng(dim + n + resident)
    rows = 2000
    host = torch.from_numpy(rng.standard_normal((rows, dim)).astype(np.float32)).pin_memory()
    ids = torch.from_numpy(rng.integers(0, rows, n).astype(np.int32)).cuda()
    ids[5::97], ids[7::89] = -1, rows
    table = torch.cat([host.cuda(), torch.zeros((1, dim), device="cuda")])
    want = table[torch.where((ids >= 0) & (ids < rows), ids.long(), torch.full_like(ids, rows).long())]
    residents = torch.from_numpy(rng.permutation(rows)[:resident].astype(np.int32))
    for staging in (2000, 300):
        c = T.cache_init(host, resident, residents, staging_rows=staging)
        for mode in (1, 0, 2):
            T.cache_tune(c, partitioned_gather=mode)
            buf = torch.full((n * dim + 40,), 7.0, device="cuda")
            out = T.cache_lookup(c, ids, out=buf[:n * dim].view(n, dim))
            assert torch.equal(out, want) and bool((buf[n * dim:] == 7.0).all()), (staging, mode)
        T.cache_free(c)


def test_lookup_replays_from_a_hip_graph_with_other_requests():
    rng = np.random.default_rng(3)
    rows, dim, n = 3000, 160, 6000
    host = torch.from_numpy(rng.standard_normal((rows, dim)).astype(np.float32)).pin_memory()
    c = T.cache_init(host, 600, None, seed=5, staging_rows=900)
    ids = torch.zeros(n, dtype=torch.int32, device="cuda")
    out = torch.empty((n, dim), dtype=torch.float32, device="cuda")
    hm = torch.zeros(2, dtype=torch.int64, device="cuda")
    T.cache_lookup(c, ids, out=out, hit_miss=hm)
    torch.cuda.synchronize()
    graph, stream = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    with torch.cuda.graph(graph, stream=stream):
        T.cache_lookup(c, ids, out=out, hit_miss=hm, stream=stream)
    for replay in range(4):
        ids_np = rng.integers(-1, rows if replay % 2 else 700, n).astype(np.int32)
        ids.copy_(torch.from_numpy(ids_np))
        hm.zero_()
        out.fill_(1.0)
        graph.replay()
        torch.cuda.synchronize()
        want = oracle.gather(host.numpy(), ids_np).tobytes()
        assert out.cpu().numpy().tobytes() == want
        hits = oracle.cache_hits(T.cache_residents(c).numpy(), rows, ids_np)
        assert tuple(hm.tolist()) == hits
        eager = T.cache_lookup(c, ids)            # the same handle, between replays
        assert eager.cpu().numpy().tobytes() == want


def test_missing_rows_in_strides_are_not_taken_for_one_popular_row():
    """3 750 rows whose ids are multiples of 16, all missing and equally popular: the launch for missed rows writes the whole
    output, tied to partitions, as for neighboring ids (132 us of that launch, and 157 where they counted as one popular row)."""
    rows, dim, n = 60_000, 413, 400_000
    host = torch.randn((rows, dim), generator=torch.Generator().manual_seed(5)).pin_memory()
    pick = torch.randint(0, rows // 16, (n,), generator=torch.Generator(device="cuda").manual_seed(8), device="cuda", dtype=torch.int32)
    c, took = T.cache_init(host, 0, staging_rows=rows), {}
    for stride in (16, 1):
        ids, out = pick * stride, torch.empty((n, dim), device="cuda")
        T.cache_lookup(c, ids, out=out)
        assert torch.equal(out, host.cuda()[ids.long()])
        took[stride] = 1e9
        for _ in range(10):
            T.profile_begin()
            T.cache_lookup(c, ids, out=out)
            took[stride] = min(took[stride], T.profile_end()["cache_gather_staged_rows"][1])
    T.cache_free(c)
    assert took[16] < 1.1 * took[1], took
