"""Parity of the forms of the epilogue with a code skip of side 0 (a table of the
scaled skip codes): with the fp32 requantisation (positive multipliers, shifts of
at least 2), where the table holds fp32 offsets that every kernel that can get the
launch has to read as such, and with the 64-bit one (shifts below 2)."""
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


# every kernel with a skip: (n, h, w, cin, cout, k, bits, bits_w)
SIDE0 = {
    "256x128": (1, 19, 23, 128, 256, 3, 4, 8),
    "256x64": (1, 67, 71, 320, 512, 1, 4, 8),
    "short": (1, 9, 11, 128, 320, 1, 4, 8),
    "stream": (1, 33, 37, 128, 256, 1, 4, 8),
    "stream_halves": (1, 25, 21, 192, 512, 1, 4, 8),
    "weight_stationary": (1, 25, 21, 256, 512, 1, 4, 8),
    "register_fed_64": (1, 93, 91, 512, 256, 1, 4, 8),
    "register_fed_64_3bit": (1, 93, 91, 512, 288, 1, 3, 8),
    "register_fed_128": (1, 115, 113, 768, 512, 1, 4, 8),
    "128x256": (1, 17, 21, 64, 128, 3, 4, 8),
    "64x512_2bit": (1, 15, 19, 64, 64, 3, 2, 4),
    "gf": (1, 15, 19, 64, 64, 3, 4, 4),
    "fx": (1, 67, 75, 1024, 512, 1, 4, 4),
    "fx3": (3, 31, 41, 256, 256, 3, 4, 4),
    "fx3_2bit": (17, 23, 19, 128, 128, 3, 2, 2),
}


@pytest.mark.parametrize("name", SIDE0)
def test_side0_skips_in_every_form(torch, name):
    """Shifts of at least 2 and positive multipliers (fp32), one negative multiplier
    (32-bit integers), shifts below 2 (64-bit integers); each launch twice, with the
    same bytes."""
    n, h, w, cin, cout, k, bits, bits_w = SIDE0[name]
    c = workloads.random_conv_case(seed=101 + cin + cout, n=n, h=h, w=w, cin=cin, cout=cout, k=k, bits_in=bits,
                                   bits_w=bits_w, wenc=workloads.WENC_TWOS, bits_out=bits, skip_bits=bits, num_levels=3)
    rng = np.random.Generator(np.random.PCG64(cin))
    for lv in c.levels:
        lv["shift"] = np.clip(lv["shift"], 2, 28).astype(np.int32)
        lv["skip_side"][:] = 0
    c.levels[1]["mult"][::7] *= -1
    c.levels[2]["shift"] = rng.integers(-2, 2, size=cout).astype(np.int32)
    c.levels[2]["mult"] = rng.integers(1 << 24, 1 << 27, size=cout).astype(np.int32)
    want = [oracle_conv(c, level) for level in range(3)]
    for _ in range(2):
        for level, got in enumerate(gpu_conv(c, torch)):
            assert_same(got, want[level], f"side 0, {name} level {level}")
