"""Parity of the handles' own kernels where a level's requantisation is done in
fp32 (positive multipliers, shifts of at least 2, code skips of side 0): the skip
table of such a launch holds fp32 offsets, which every kernel that can get the
launch has to read as such."""
import numpy as np
import pytest

from gpu_helpers import assert_same, gpu_conv, oracle_conv
from paper_2007_06919_amd import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available()
    return t


# (n, h, w, cin, cout, k, bits, bits_w, skip, up2). 8-bit weights: no block-float
# form, the handle's own kernel at any size
SHORT = [
    # up to 4 K steps, channels that are not a multiple of 256: 256 x 64 tiles, three to a CU
    (1, 83, 85, 64, 320, 1, 4, 4, 4, False),
    (2, 61, 77, 192, 288, 1, 3, 3, 3, False),
    (1, 83, 85, 256, 320, 1, 4, 4, 4, True),
    (1, 9, 11, 128, 320, 1, 4, 8, 4, False),
    (1, 9, 11, 128, 320, 1, 4, 8, 0, False),
    (3, 1, 1, 64, 288, 1, 4, 8, 4, False),
]


@pytest.mark.parametrize("case", SHORT, ids=lambda c: "x".join(map(str, c)))
def test_short_tiles(torch, case):
    n, h, w, cin, cout, k, bits, bits_w, skip, up2 = case
    c = workloads.random_conv_case(seed=97 + cin, n=n, h=h, w=w, cin=cin, cout=cout, k=k, bits_in=bits, bits_w=bits_w,
                                   wenc=workloads.WENC_TWOS, bits_out=bits, skip_bits=skip, skip_up2=up2)
    lv = c.levels[0]
    lv["shift"] = np.clip(lv["shift"], 2, 28).astype(np.int32)
    if skip:
        lv["skip_side"][:] = 0
    assert_same(gpu_conv(c, torch)[0], oracle_conv(c), f"short tiles {case}")
