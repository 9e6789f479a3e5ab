"""The native half of the Python binding against the general (ctypes) half, over the forms both accept, and its refusals."""
import numpy as np
import pytest
import torch

import paper_2402_05396_amd as T

pytestmark = pytest.mark.gpu


class _Absent:
    """Takes no call: every function of the binding then goes its general way."""

    def __getattr__(self, name):
        return lambda *a: None


class _Subclass(torch.Tensor):
    pass


def _graph(n=5000, nodes=300):
    rng = np.random.default_rng(4)
    d = lambda a: torch.from_numpy(a).cuda()
    src, dst = rng.integers(0, nodes, (2, n)).astype(np.int32)
    ts = np.sort(rng.integers(0, 2000, n)).astype(np.int64)
    g = T.tcsr_build(d(src), d(dst), d(ts), None, nodes)
    return g, d(rng.integers(-1, nodes, 200).astype(np.int32)), d(rng.integers(0, 2100, 200).astype(np.int64)), rng


def _same(a, b):
    if isinstance(a, dict):
        assert list(a) == list(b)
        return all(_same(a[k], b[k]) for k in a)
    if isinstance(a, (list, tuple)):
        assert type(a) is type(b) and len(a) == len(b)
        return all(_same(x, y) for x, y in zip(a, b))
    if a is None or b is None:
        return a is b
    assert a.dtype == b.dtype and a.shape == b.shape and a.device == b.device and a.is_contiguous(), (a.shape, b.shape)
    return torch.equal(a, b)


def test_both_halves_give_the_same(monkeypatch):
    g, roots, times, rng = _graph()
    table = torch.randn((5000, 20), device="cuda")
    half = torch.randn((5000, 40), device="cuda", dtype=torch.float16)[:, 1:38]
    weight = torch.randint(1, 99, (5000,), device="cuda", dtype=torch.int32)
    side = torch.cuda.Stream()
    host = torch.randn((300, 9)).pin_memory()
    cache = T.cache_init(host, 50, None, staging_rows=100)
    selector = T.selector_init(n=4000, initial_score=3)
    cand = T.sample_temporal(g, roots, times, 25, 1, T.RECENT, 0)[0]
    w = torch.randint(1, 99, (200, 25), device="cuda", dtype=torch.int32)
    ids = torch.randint(-1, 300, (1000,), device="cuda", dtype=torch.int32)
    side.wait_stream(torch.cuda.current_stream())
    calls = []
    for policy in range(4):
        for hops in (1, 2):
            for stream in (None, side):
                calls.append(lambda p=policy, h=hops, s=stream: T.sample_temporal(g, roots, times, 5, h, p, 2 ** 64 - 3, 20, weight, stream=s))
                calls.append(lambda p=policy, h=hops, s=stream: T.sample_temporal_rows(g, roots, times, 5, h, p, -7, table, 20, weight, stream=s))
        calls.append(lambda p=policy: T.sample_temporal_rows(g, roots[:0], times[:0], 5, 2, p, 1, half, 20, weight))
        calls.append(lambda p=policy: T.sample_temporal_rows(g, roots, times, 3, 2, p, 1, half, 20, weight, row_elems=11))
    calls += [lambda: T.gather_features(half, ids), lambda: T.gather_features(table, ids, row_elems=3, stream=side),
              lambda: T.gather_features(table, ids, out=torch.empty(21_000, device="cuda"))[:20_000], lambda: T.gather_features(table, ids[:0]),
              lambda: T.candidate_encodings(cand["nbr"], cand["count"]), lambda: T.candidate_encodings(cand["nbr"], cand["count"], False, side),
              lambda: T.select_weighted(w, cand["count"], 10, 5, 1), lambda: T.select_weighted(w, cand["count"], 10, 5, 2 ** 32 - 1, cand),
              lambda: T.cache_lookup(cache, ids), lambda: T.cache_lookup(cache, ids, hit_miss=torch.zeros(2, dtype=torch.int64, device="cuda")),
              lambda: T.cache_lookup(cache, ids, out=torch.empty((1000, 9), device="cuda"), stream=side),
              lambda: (T.selector_update(selector, ids[:50].abs(), ids[50:100].abs()), T.selector_scores(selector, want_total=False)),
              lambda: T.selector_draw(selector, 30, 7, 2 ** 40), lambda: T.selector_draw(selector, 0, 7, 1),
              lambda: T.selector_draw(selector, 30, 7, 4, out=torch.empty(40, dtype=torch.int32, device="cuda"))[:30]]
    native = []
    for call in calls:
        native.append(call())
        torch.cuda.synchronize()
    monkeypatch.setattr(T, "_native", _Absent())
    for i, (call, a) in enumerate(zip(calls, native)):
        b = call()
        torch.cuda.synchronize()
        assert _same(a, b), i


def test_what_was_refused_stays_refused():
    g, roots, times, _ = _graph()
    table = torch.randn((5000, 20), device="cuda")
    ids = torch.zeros(8, dtype=torch.int32, device="cuda")
    for bad in (roots.long(), roots.cpu(), roots[::2]):
        with pytest.raises((TypeError, ValueError)):
            T.sample_temporal(g, bad, times, 5, 1, T.RECENT, 0)
        with pytest.raises(TypeError):
            T.gather_features(table, bad)
    with pytest.raises(ValueError):
        T.sample_temporal(g, roots, times[:-1], 5, 1, T.RECENT, 0)
    for k, hops, policy, m, code in ((0, 1, 0, 0, -2), (65, 1, 0, 0, -2), (5, 4, 0, 0, -2), (5, 0, 0, 0, -2), (5, 1, 9, 0, -1), (5, 1, T.WEIGHTED, 5, -1)):
        with pytest.raises(T.TaserError) as e:
            T.sample_temporal(g, roots, times, k, hops, policy, 0, m)
        assert e.value.code == code and str(code) in str(e.value)
    with pytest.raises(TypeError):
        T.gather_features(table.t(), ids)
    with pytest.raises(TypeError):
        T.gather_features(table, ids, out=torch.empty(3, device="cuda"))
    with pytest.raises(TypeError):
        T.gather_features(table.cpu(), ids)
    with pytest.raises(ValueError):
        T.candidate_encodings(ids.view(2, 4), ids[:3])
    g.free()
    with pytest.raises(T.TaserError):
        T.sample_temporal(g, roots, times, 5, 1, T.RECENT, 0)


def test_other_tensor_types_take_the_general_way():
    g, roots, times, _ = _graph()
    a = T.sample_temporal(g, roots, times, 5, 2, T.UNIFORM, 3)
    b = T.sample_temporal(g, roots.as_subclass(_Subclass), times, np.int64(5), 2, T.UNIFORM, 3)
    assert _same([{k: v.as_subclass(torch.Tensor) for k, v in h.items()} for h in b], a)
