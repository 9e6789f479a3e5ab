"""Candidate encodings where a block's identity bytes begin and end inside a 16-byte piece, or a window is a block's only one, and
around the size from which odd windows are written past the caches."""
import numpy as np
import pytest
import torch

import oracle
import paper_2402_05396_amd as T

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [1, 7, 15, 16, 17, 25, 31, 32, 33, 49, 63, 64])
@pytest.mark.parametrize("roots", [1, 3, 4, 5, 15, 16, 17, 31, 33, 200])
@pytest.mark.parametrize("shift", [0, 4, 13])
def test_encodings(m, roots, shift):
    rng = np.random.default_rng(m * 1000 + roots)
    nbr, count = rng.integers(0, max(2, m // 2), (roots, m)).astype(np.int32), rng.integers(0, m + 1, roots).astype(np.int32)
    want_f, want_i = oracle.candidate_encodings(nbr, count)
    d_nbr, d_count = torch.from_numpy(nbr).cuda(), torch.from_numpy(count).cuda()
    freq = torch.empty((roots, m), dtype=torch.int32, device="cuda")
    buf = torch.full((shift + roots * m * m + 40,), 9, dtype=torch.uint8, device="cuda")
    view = buf[shift:]
    T._check(T.lib().taser_candidate_encodings(T._ptr(d_nbr), T._ptr(d_count), roots, m, T._ptr(freq), T._ptr(view), None))
    torch.cuda.synchronize()
    assert np.array_equal(freq.cpu().numpy(), want_f)
    assert np.array_equal(view[:roots * m * m].cpu().numpy().reshape(roots, m, m), want_i)
    assert bool((buf[:shift] == 9).all()) and bool((view[roots * m * m:] == 9).all())


@pytest.mark.parametrize("m", [7, 15, 17, 31, 33, 63])
@pytest.mark.parametrize("above", [False, True])
def test_odd_windows_around_twelve_megabytes(m, above):
    rng = np.random.default_rng(m)
    roots = -(-(12 << 20) // (m * m)) - (0 if above else 1)
    nbr, count = rng.integers(0, max(2, m // 2), (roots, m)).astype(np.int32), rng.integers(0, m + 1, roots).astype(np.int32)
    want_f, want_i = oracle.candidate_encodings(nbr, count)
    freq, identity = T.candidate_encodings(torch.from_numpy(nbr).cuda(), torch.from_numpy(count).cuda())
    assert np.array_equal(freq.cpu().numpy(), want_f) and np.array_equal(identity.cpu().numpy().reshape(want_i.shape), want_i)
