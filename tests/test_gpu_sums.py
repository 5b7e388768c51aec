"""Exact per-channel sums of an int32 tensor (aqd_channel_sums) against numpy:
the 16-byte form (channel counts that are a multiple of 4, aligned tensors) and
the general one, strips shorter than a row group, one row, many rows, values at
the ends of int32."""
import numpy as np
import pytest

from paper_2007_06919_amd import aqd

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows, c, shift", [(1, 4, 0), (3, 256, 0), (33, 260, 0), (4097, 36, 0), (70000, 64, 0),
                                            (257, 1024, 0), (515, 256, 1), (100, 7, 0)])
def test_channel_sums_forms(rows, c, shift):
    """shift: the tensor starts that many int32 past an aligned address."""
    import torch
    rng = np.random.Generator(np.random.PCG64(rows + c))
    v = rng.integers(-(1 << 31), (1 << 31) - 1, size=(rows, c)).astype(np.int32) >> (8 if rows > 1000 else 4)
    buf = torch.zeros(rows * c + shift, dtype=torch.int32, device="cuda:0")
    buf[shift:] = torch.from_numpy(v.ravel()).cuda()
    sums = torch.full((2 * c,), 5, dtype=torch.int64, device="cuda:0")   # accumulated into
    for _ in range(2):
        aqd.channel_sums(buf.data_ptr() + 4 * shift, rows, c, sums)
    torch.cuda.synchronize()
    w = v.astype(np.int64)
    want = np.concatenate([w.sum(0), (w * w).sum(0)]) * 2 + 5
    assert np.array_equal(sums.cpu().numpy(), want)
