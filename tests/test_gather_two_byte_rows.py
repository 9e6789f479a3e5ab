"""Gathers of rows that are only 2-byte aligned, at the edges of the 16-byte pieces and of the blocks."""
import numpy as np
import pytest
import torch

import oracle
import paper_2402_05396_amd as T

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim,pitch,offset,n", [
    (7, 7, 0, 1000),            # 14 bytes: shorter than a piece, the element kernel
    (8, 9, 0, 1025), (8, 8, 1, 4099), (9, 9, 0, 1), (9, 9, 0, 7), (9, 11, 1, 5000),
    (15, 15, 1, 3001), (16, 17, 1, 2049), (17, 17, 0, 3000), (23, 24, 1, 999),
    (413, 413, 0, 20_003), (413, 415, 1, 79), (8191, 8191, 0, 33), (8192, 8193, 1, 5),
    (61_001, 61_001, 0, 9), (65_537, 65_537, 0, 5),   # rows on both sides of where the division by a multiply is exact
    # the same from where the 16-byte pieces take over: 32 MiB of short rows, 1 MiB of rows of whole pieces, 4 MiB of others
    (8, 9, 0, (1 << 21) + 1), (9, 9, 1, 1_864_136), (15, 15, 1, 1_200_001), (17, 17, 0, 999_999), (23, 24, 1, 730_003), (27, 28, 0, 621_379),
    (16, 17, 1, 32_767), (16, 16, 1, 32_769), (40, 41, 0, 30_001), (28, 29, 1, 74_899), (28, 28, 1, 74_900), (33, 33, 1, 63_551), (413, 415, 1, 5079),
    (8191, 8191, 0, 257), (8192, 8193, 1, 255), (61_001, 61_001, 0, 35), (65_537, 65_537, 0, 33),
])
def test_two_byte_rows_equal_the_oracle(dim, pitch, offset, n):
    rng = np.random.default_rng(dim * 31 + n)
    rows = max(3, min(500, 4_000_000 // pitch))
    flat = torch.from_numpy(rng.integers(-2 ** 15, 2 ** 15, offset + rows * pitch + 8, dtype=np.int16)).cuda()
    table = flat[offset:offset + rows * pitch].view(rows, pitch)
    ids = rng.integers(-1, rows + 1, n).astype(np.int32)         # padding and ids beyond the table among them
    ids[-1] = rows - 1                                           # the table's very last bytes
    guard = torch.full((n * dim + 64,), 0x1234, dtype=torch.int16, device="cuda")
    out = T.gather_features(table, torch.from_numpy(ids).cuda(), out=guard[:n * dim], row_elems=dim)
    want = oracle.gather(np.ascontiguousarray(table.cpu().numpy()[:, :dim]), np.where(ids >= rows, -1, ids))
    assert out.cpu().numpy().tobytes() == want.tobytes()
    assert bool((guard[n * dim:] == 0x1234).all())
