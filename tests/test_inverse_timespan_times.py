"""Times of the inverse-timespan finder that tell one rule of its kernel from another: ratios of calls made in turn."""
import numpy as np
import pytest
import torch

import paper_2402_05396_amd as T


def _call(entries, nodes, span, roots, k):
    """Lists of equal length, timestamps spread evenly over the span, queries from its second half."""
    rng = np.random.default_rng(nodes)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    src = (np.arange(entries) % nodes).astype(np.int32)
    g = T.tcsr_build(dev(src), dev(src), dev(np.sort(rng.integers(0, span, entries)).astype(np.int64)), None, nodes)
    q, t = dev(rng.integers(0, nodes, roots).astype(np.int32)), dev(rng.integers(span // 2, span, roots).astype(np.int64))
    out = T.sample_outputs(roots, k, 1, "cuda")
    return lambda: T.sample_temporal(g, q, t, k, 1, T.INVERSE_TIMESPAN, 5, out=out)


def _ratio(a, b):
    """Time of a over time of b, the best of twelve turns of twenty calls each."""
    begin, end, best = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True), [1e9, 1e9]
    for _ in range(13):
        for i, f in enumerate((a, b)):
            f()
            begin.record()
            for _ in range(20):
                f()
            end.record()
            end.synchronize()
            best[i] = min(best[i], begin.elapsed_time(end))
    print([round(x * 50, 1) for x in best])
    return best[0] / best[1]


@pytest.mark.gpu
def test_blocks_of_one_root_leave_room_for_others():
    """2 000 blocks are resident at once; of 3 000 the last thousand wait for room, but not for more than LDS takes: 1.33
    times as long (1.68 with the LDS of four roots in each)."""
    assert _ratio(_call(1_000_000, 3000, 1 << 28, 3000, 10), _call(1_000_000, 3000, 1 << 28, 2000, 10)) < 1.5


@pytest.mark.gpu
def test_many_draws_are_not_made_from_weights():
    """64 draws from lists of 3 300 entries, few per weight: about as long where the timestamps spread over 2^31 ticks as where
    they leave no weight with several entries (1.3 times with a list summed by weights, whatever the draws)."""
    assert _ratio(_call(1_000_000, 300, 1 << 31, 4000, 64), _call(1_000_000, 300, 1 << 24, 4000, 64)) < 1.15
