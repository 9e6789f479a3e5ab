"""Calls of the library that allocate, where the driver's memory is taken up by blocks that torch keeps."""
import types

import pytest
import torch

import paper_2402_05396_amd as T


class _Full:
    """Stands in for libtaser.so: every entry point is out of memory until torch's blocks are given back `after` times."""

    def __init__(self, after):
        self.after, self.given_back, self.calls = after, 0, []

    def __getattr__(self, name):
        def entry(*args):
            self.calls.append(name)
            return 0 if self.given_back >= self.after else -3
        return entry

    def taser_last_error(self):
        return b"no memory"

    def give_back(self):
        self.given_back += 1


@pytest.mark.parametrize("after", [0, 1, 2])
def test_blocks_that_torch_keeps_are_given_back_before_a_call_fails(monkeypatch, after):
    stream = types.SimpleNamespace(cuda_stream=0)
    cache = types.SimpleNamespace(handle=None)
    host = torch.zeros((4, 4))
    for name, call in (("taser_selector_init", lambda: T.selector_init(n=10, stream=stream)),
                       ("taser_cache_init", lambda: T.cache_init(host, 2, staging_rows=3, stream=stream)),
                       ("taser_cache_count_accesses", lambda: T.cache_count_accesses(cache, stream=stream))):
        full = _Full(after)
        monkeypatch.setattr(T, "_lib", full)
        monkeypatch.setattr(torch.cuda, "empty_cache", full.give_back)
        if after < 2:
            call()
        else:
            with pytest.raises(T.TaserError) as e:
                call()
            assert e.value.code == -3
        assert full.calls[:2] == [name] * min(2, after + 1) and full.given_back == min(1, after)


@pytest.mark.gpu
def test_calls_without_outputs_of_the_callers_reach_the_second_attempt(monkeypatch):
    """The native half leaves a call that ran out of memory to the general one, which makes it again."""
    d = lambda *a: torch.tensor(a, device="cuda")
    g = T.tcsr_build(d(0, 1).int(), d(1, 0).int(), d(3, 4), None, 2)
    cache = T.cache_init(torch.ones((4, 4)).pin_memory(), 2)
    roots, times = d(0, 1).int(), d(9, 9)
    want = T.sample_temporal(g, roots, times, 2, 1, T.INVERSE_TIMESPAN, 1)[0]["nbr"]
    T.cache_lookup(cache, roots)                       # binds the native half to the real library
    real, full = T._lib, _Full(1)
    import ctypes
    failing = ctypes.CFUNCTYPE(ctypes.c_int)(lambda: -3)
    addresses = {n: ctypes.cast(getattr(real, n), ctypes.c_void_p).value for n in T.EXPORTS}
    for n in ("taser_sample_temporal", "taser_sample_temporal_rows", "taser_cache_lookup"):
        addresses[n] = ctypes.cast(failing, ctypes.c_void_p).value
    T._native.bind(T.TaserError, addresses)
    try:
        assert torch.equal(T.sample_temporal(g, roots, times, 2, 1, T.INVERSE_TIMESPAN, 1)[0]["nbr"], want)
        _, rows = T.sample_temporal_rows(g, roots, times, 2, 1, T.RECENT, 1, torch.ones((2, 4), device="cuda"))
        assert rows[0].shape == (4, 4)
        assert torch.equal(T.cache_lookup(cache, roots), torch.ones((2, 4), device="cuda"))
        monkeypatch.setattr(T, "_lib", full)
        monkeypatch.setattr(torch.cuda, "empty_cache", full.give_back)
        T.sample_temporal(g, roots, times, 2, 1, T.RECENT, 1)
        assert full.calls == ["taser_sample_temporal"] * 2 and full.given_back == 1
    finally:
        monkeypatch.setattr(T, "_lib", real)
        T._bind()
