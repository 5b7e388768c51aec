"""Parity of the global-fed kernel (operands straight from global memory, the
waves of a tile splitting its K range) against the oracle, bit for bit: every
tile and split its rule picks (64 x 64 tiles on 1, 2 and 4 waves, 64 x 32 and
32 x 32 on 4, 16 channels x 64 pixels for at most 4 channels), the three operand formats,
every output and skip width, steps that span taps, partial channel groups and
pixel tiles, and sums at the bound where fp32 stops being exact."""
import numpy as np
import pytest

from gpu_helpers import assert_same, check_case, gpu_conv, oracle_conv
from oracle import ref
from paper_2007_06919_amd import aqd, workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available()
    return t


CASES = {
    # <= 64 tiles of 64 x 64: 32 x 32, <= 100: 64 x 32 (the second case), 4 waves
    "f6_k5_two_taps_a_step": dict(n=1, h=32, w=32, cin=64, cout=64, k=3),
    "f6_64x32": dict(n=1, h=25, w=42, cin=256, cout=256, k=3, skip_bits=4, wenc=1),
    "f6_up2_skip": dict(n=2, h=13, w=21, cin=256, cout=256, k=3, skip_bits=4, skip_up2=True, wenc=1),
    "f6_cin96_partial_group_int32": dict(n=1, h=9, w=11, cin=96, cout=80, k=3, stride=2, bits_out=32, wenc=1),
    "f6_cin32_one_step": dict(n=1, h=9, w=11, cin=32, cout=36, k=1, bits_out=32),
    "f6_cout20_kernel5": dict(n=1, h=17, w=5, cin=64, cout=20, k=5),
    "f6_int32_skip": dict(n=1, h=17, w=5, cin=128, cout=256, k=1, skip_bits=32, wenc=1),
    "f6_8bit_out": dict(n=2, h=7, w=11, cin=256, cout=256, k=3, bits_out=8, wenc=1),
    "f6_3bit_levels": dict(n=2, h=7, w=11, cin=64, cout=64, k=3, bits_in=3, bits_w=3, bits_out=3, skip_bits=3,
                           wenc=1, num_levels=2),
    "f4_skip": dict(n=1, h=9, w=11, cin=128, cout=128, k=3, bits_in=2, bits_w=2, bits_out=2, skip_bits=2, wenc=1),
    "i8_int32": dict(n=2, h=7, w=11, cin=128, cout=36, k=3, bits_in=8, bits_w=8, bits_out=32),
    "i8_8bit_out_skip": dict(n=2, h=7, w=11, cin=48, cout=40, k=3, bits_in=8, bits_w=4, bits_out=8, skip_bits=8),
    "i8_int32_skip_cin16": dict(n=1, h=7, w=11, cin=16, cout=12, k=3, bits_in=8, bits_w=8, bits_out=4, skip_bits=32),
    # 1 to 4 channels
    "f6_cout1": dict(n=2, h=13, w=21, cin=256, cout=1, k=3, bits_out=32, wenc=1),
    "f6_cout3": dict(n=2, h=7, w=9, cin=64, cout=3, k=1, bits_out=32, wenc=1),
    "f6_cout4_codes": dict(n=2, h=13, w=21, cin=64, cout=4, k=3),
    "f4_cout2_long_k": dict(n=2, h=13, w=21, cin=2048, cout=2, k=3, bits_in=2, bits_w=2, bits_out=32),
    # 101 - 400 tiles: 64 x 64, 4 waves (2 steps: 2 waves)
    "f6_4waves": dict(n=1, h=50, w=45, cin=256, cout=256, k=3, wenc=1),
    "f6_1x1_two_steps": dict(n=1, h=50, w=45, cin=256, cout=128, k=1, skip_bits=4),
    # 401 - 1000 tiles: 2 waves; more: 1 wave
    "f6_2waves_int32": dict(n=1, h=89, w=133, cin=128, cout=132, k=3, bits_out=32, wenc=1),
    "f6_1wave": dict(n=1, h=179, w=361, cin=64, cout=64, k=3, wenc=1),
    "f4_1wave_stride2": dict(n=2, h=181, w=339, cin=64, cout=192, k=3, stride=2, bits_in=2, bits_w=2, bits_out=2),
}


# tiled kernel: 256 x 128, 256 x 64 and 128 x 128 tiles, stages that span taps
# (cin 32 to 96) or end in the middle (odd step counts), partial channel tiles
# (more than one group past the last), ragged pixel tiles, skips of mixed and
# zero sides, the 64-bit requantisation (shifts below 2)
TILED = {
    "f6_256x128": dict(n=2, h=193, w=181, cin=256, cout=256, k=3, stride=2, wenc=1),
    "f6_256x128_partial_cout": dict(n=1, h=97, w=91, cin=160, cout=592, k=3, wenc=1),
    "f6_256x128_int32": dict(n=1, h=75, w=91, cin=160, cout=720, k=3, bits_out=32, wenc=1),
    "f6_256x64": dict(n=1, h=67, w=75, cin=1024, cout=512, k=1),
    "f6_256x64_skip_cin160": dict(n=1, h=83, w=75, cin=160, cout=512, k=3, skip_bits=4),
    "f6_256x64_3bit": dict(n=1, h=83, w=75, cin=192, cout=384, k=3, bits_in=3, bits_w=3, bits_out=3, wenc=1),
    "f6_128x128_int32": dict(n=2, h=131, w=141, cin=160, cout=80, k=3, bits_out=32, wenc=1),
    "f6_128x128_stride2": dict(n=2, h=261, w=251, cin=128, cout=128, k=3, stride=2, wenc=1),
    "f4_256x128": dict(n=2, h=299, w=331, cin=32, cout=256, k=3, bits_in=2, bits_w=2, bits_out=2, wenc=1),
    "f4_256x64_skip_up2": dict(n=1, h=83, w=75, cin=256, cout=512, k=1, bits_in=2, bits_w=2, bits_out=2, skip_bits=2,
                               skip_up2=True),
    "f4_256x128_int32": dict(n=1, h=201, w=203, cin=96, cout=516, k=3, bits_in=2, bits_w=2, bits_out=32, wenc=1),
    "f4_128x128": dict(n=2, h=131, w=141, cin=96, cout=112, k=3, bits_in=2, bits_w=2, bits_out=2, skip_bits=2),
    # 1x1 layers of 2 bits: 128 x 128 tiles with partial ones at the end of the
    # channels (320 = 2 1/2 tiles), skips and int32 outputs on many pixels; own tiles
    # for 64 channels on many pixels
    "f4_128x128_320": dict(n=1, h=131, w=141, cin=128, cout=320, k=1, bits_in=2, bits_w=2, bits_out=2, wenc=1),
    "f4_128x128_320_skip": dict(n=1, h=131, w=141, cin=192, cout=320, k=1, bits_in=2, bits_w=2, bits_out=2, skip_bits=2,
                                skip_up2=True),
    "f4_128x128_256_int32": dict(n=1, h=183, w=191, cin=64, cout=260, k=1, bits_in=2, bits_w=2, bits_out=32, wenc=1),
    "f4_own_64": dict(n=1, h=263, w=271, cin=64, cout=64, k=1, bits_in=2, bits_w=2, bits_out=2, skip_bits=2),
    # 3x3 stride 1 with the tile's input in LDS: every block size (64, 128, 256
    # channels, two blocks), tiles that span rows, images and pads (rows shorter
    # than a tile), partial channel tiles; images on either side of the share of
    # padding up to which this kernel runs, and of more than 256 channels to few
    "fx3_cin64": dict(n=3, h=61, w=77, cin=64, cout=64, k=3, wenc=1),
    "fx3_cin64_skip_3bit": dict(n=3, h=61, w=77, cin=64, cout=80, k=3, bits_in=3, bits_w=3, bits_out=3, skip_bits=3),
    "fx3_cin64_int32": dict(n=40, h=23, w=15, cin=64, cout=36, k=3, bits_out=32, wenc=1),
    "fx3_cin128": dict(n=17, h=23, w=19, cin=128, cout=128, k=3, wenc=1),
    "fx3_cin128_skip": dict(n=17, h=23, w=19, cin=128, cout=112, k=3, wenc=1, skip_bits=4),
    "fx3_cin256_256x64": dict(n=3, h=31, w=41, cin=256, cout=256, k=3, wenc=1),
    "fx3_cin256_256x128": dict(n=9, h=41, w=47, cin=256, cout=272, k=3, wenc=1),
    "fx3_cin256_128x128_skip": dict(n=9, h=21, w=47, cin=256, cout=256, k=3, wenc=1, skip_bits=4),
    "fx3_cin256_256x64_skip": dict(n=9, h=51, w=57, cin=256, cout=256, k=3, wenc=1, skip_bits=4),
    "fx3_cin256_int32": dict(n=5, h=41, w=47, cin=256, cout=324, k=3, bits_out=32, wenc=1),
    "fx3_cin256_narrow_int32": dict(n=9, h=41, w=47, cin=256, cout=80, k=3, bits_out=32, wenc=1),
    "fx3_cin512_skip": dict(n=3, h=25, w=27, cin=512, cout=528, k=3, skip_bits=4),
    "fx3_1x1_images": dict(n=3500, h=1, w=1, cin=256, cout=256, k=3, wenc=1),
    "fx3_2x300": dict(n=7, h=2, w=300, cin=128, cout=256, k=3, wenc=1),
    "fx3_4x5_images": dict(n=700, h=4, w=5, cin=128, cout=128, k=3, wenc=1),
    "fx3_8x9_images_skip": dict(n=130, h=8, w=9, cin=256, cout=256, k=3, wenc=1, skip_bits=4),
    "too_much_padding_3x4_images": dict(n=900, h=3, w=4, cin=64, cout=64, k=3, wenc=1),
    "too_much_padding_7x8_images": dict(n=170, h=7, w=8, cin=256, cout=256, k=3, wenc=1),
    "f6_128x128_cin512": dict(n=5, h=61, w=77, cin=512, cout=112, k=3, wenc=1, skip_bits=4),
    "f6_256x64_cin512_192": dict(n=4, h=3, w=1200, cin=512, cout=192, k=3, wenc=1, skip_bits=4),
    "f6_256x128_cin512_144": dict(n=1, h=2, w=24000, cin=512, cout=144, k=3, bits_in=3, bits_w=2, bits_out=3),
    "f4_128x128_cin512": dict(n=5, h=61, w=77, cin=512, cout=128, k=3, bits_in=2, bits_w=2, bits_out=2, wenc=1),
    "fx3_f4_cin64": dict(n=3, h=61, w=77, cin=64, cout=64, k=3, bits_in=2, bits_w=2, bits_out=2, wenc=1, skip_bits=2),
    "fx3_f4_cin128": dict(n=17, h=23, w=19, cin=128, cout=128, k=3, bits_in=2, bits_w=2, bits_out=2),
    "fx3_f4_cin256": dict(n=3, h=61, w=77, cin=256, cout=272, k=3, bits_in=2, bits_w=2, bits_out=2, skip_bits=2),
    "fx3_f4_cin256_int32": dict(n=2, h=91, w=97, cin=256, cout=720, k=3, bits_in=2, bits_w=2, bits_out=32, wenc=1),
    "fx3_f4_cin512": dict(n=3, h=25, w=27, cin=512, cout=512, k=3, bits_in=2, bits_w=2, bits_out=2, wenc=1),
}


@pytest.mark.parametrize("name", TILED)
def test_tiled_parity(torch, name):
    check_case(torch, seed=800 + len(name), **TILED[name])


@pytest.mark.parametrize("bits, skip", [(4, 0), (4, 4), (2, 0), (2, 2)])
def test_tiled_epilogue_forms(torch, bits, skip):
    """64-bit requantisation (a shift below 2), and skips whose sides are all 0
    (the table of scaled codes)."""
    for form in ("slow", "side0", "slow 3x3", "side0 3x3"):
        case = workloads.random_conv_case(seed=61 + bits, n=1, h=83, w=75, cin=256 if "3x3" in form else 160, cout=512,
                                          k=3, bits_in=bits, bits_w=bits, bits_out=bits, skip_bits=skip)
        lv = case.levels[0]
        if "slow" in form:
            lv["shift"][5] = 1
            lv["mult"][5] = 1 << 30
        elif skip:
            lv["skip_side"][:] = 0
        assert_same(gpu_conv(case, torch)[0], oracle_conv(case), f"{bits}-bit {form}")


@pytest.mark.parametrize("name", CASES)
def test_global_fed_parity(torch, name):
    check_case(torch, seed=700 + len(name), **CASES[name])


@pytest.mark.parametrize("bits, cin, k", [(4, 8192, 3), (3, 16384, 3), (2, 16384, 5)])
def test_sums_at_the_exact_bound(torch, bits, cin, k):
    """All weights at the largest odd-grid value, all codes at the largest
    but a few 1s (and some negative weights in the second channel half): sums up
    to K * (2^b - 1)^2, just below 2^24 at 4 bits, exact in every term order."""
    q = (1 << bits) - 1
    assert cin * k * k * q * q < 1 << 24
    case = workloads.random_conv_case(seed=31 + bits, n=1, h=5, w=6, cin=cin, cout=64, k=k, bits_in=bits,
                                      bits_w=bits, wenc=1, bits_out=32)
    rng = np.random.Generator(np.random.PCG64(bits))
    case.x[:] = q
    case.x[rng.random(case.x.shape) < 0.01] = 1
    case.w_fields[:] = q
    case.w_fields[32:][rng.random(case.w_fields[32:].shape) < 0.05] = 0
    assert_same(gpu_conv(case, torch)[0], oracle_conv(case), f"{bits}-bit sums near 2^24")


# 8-bit codes: (n, h, w, cin, cout, bits_out), the tiles and splits of the int8
# form (32 x 32, 64 x 32 and 64 x 64 on 4 waves, 64 x 64 on 2 and on 1, 16
# channels x 64 pixels for at most 4 channels)
I8_SUMS = [(1, 9, 11, 256, 128, 32), (1, 9, 11, 144, 72, 8), (1, 25, 41, 256, 256, 32), (1, 50, 45, 256, 128, 32),
           (1, 50, 45, 144, 256, 8), (1, 150, 201, 144, 8, 32), (1, 150, 201, 144, 8, 8), (1, 250, 270, 144, 8, 32),
           (1, 13, 21, 144, 4, 32), (1, 13, 21, 144, 4, 8), (1, 13, 21, 256, 3, 32)]


@pytest.mark.parametrize("case", I8_SUMS, ids=lambda c: "x".join(map(str, c)))
def test_eight_bit_sums_past_the_fp32_integers(torch, case):
    """Codes 255 and weights 127 or -127 but for a few 254s and 126s: the
    re-centred sums are odd as well as even and beyond 2^24, where fp32 holds even
    numbers only. Code outputs: a requantisation of scale 1 whose bias puts each
    channel's interior sums within the code range, so that a sum off by one shows."""
    n, h, w, cin, cout, bits_out = case
    c = workloads.random_conv_case(seed=41, n=n, h=h, w=w, cin=cin, cout=cout, k=3, bits_in=8, bits_w=8,
                                   bits_out=bits_out)
    K = 9 * cin
    rng = np.random.Generator(np.random.PCG64(K))
    c.x[:] = np.where(rng.random(c.x.shape) < 1 / K, 254, 255)
    wv = np.where(rng.random(c.w_fields.shape) < 0.01, 126, 127) * np.where(np.arange(cout) % 2, -1, 1).reshape(-1, 1, 1, 1)
    c.w_fields[:] = wv & 0xFF
    sums = wv.reshape(cout, -1).sum(1)
    lv = c.levels[0]
    if bits_out == 8:   # interior sums are 255 * sum(w) less about one |w|
        lv["bias"] = (-255 * sums + np.where(sums > 0, 255, 0)).astype(np.int32)
        lv["mult"][:], lv["shift"][:] = 1 << 30, -1
    want = oracle_conv(c)
    if bits_out == 32:
        recentred = want.astype(np.int64) - lv["bias"] - 128 * sums
        lost = recentred != recentred.astype(np.float32).astype(np.int64)
        assert lost.mean() > 0.2, "the sums do not pass what fp32 holds"
    else:
        assert ((want > 0) & (want < 255)).mean() > 0.2
    assert_same(gpu_conv(c, torch)[0], want, f"8-bit sums past 2^24 {case}")


@pytest.mark.parametrize("wenc", [workloads.WENC_TWOS, workloads.WENC_PAPER_ODD])
@pytest.mark.parametrize("shape", [(1, 9, 11, 64, 64, 3), (3, 61, 77, 64, 64, 3), (1, 67, 75, 1024, 512, 1)],
                         ids=["gf", "fx3", "fx"])
def test_three_bit_weights_with_the_spare_bit_set(torch, shape, wenc):
    """A 3-bit weight field is the low three bits of its 4-bit container: the
    fourth may hold anything, such as a copy of the sign."""
    n, h, w, cin, cout, k = shape
    case = workloads.random_conv_case(seed=83, n=n, h=h, w=w, cin=cin, cout=cout, k=k, bits_in=3, bits_w=3, bits_out=3,
                                      wenc=wenc)
    packed = aqd.pack_codes(case.w_fields, 3)
    spare = np.random.Generator(np.random.PCG64(84)).integers(0, 256, size=packed.shape, dtype=np.uint8) & 0x88
    if wenc == workloads.WENC_TWOS:
        spare = (packed & 0x44) << 1   # sign extended
    assert spare.any()
    assert_same(gpu_conv(case, torch, w_packed=packed | spare)[0], oracle_conv(case), "3-bit weights, spare bit set")


def test_grouped_levels_of_small_images(torch):
    """One 3x3 launch over levels whose last images are narrower than the filter:
    the padding rows and columns of neighbouring images fall into one tile."""
    sizes = [(41, 47), (9, 11), (2, 3), (1, 1), (1, 5)]
    case = workloads.random_conv_case(seed=93, n=1, h=8, w=8, cin=256, cout=256, k=3, wenc=1, num_levels=len(sizes))
    handle = aqd.qconv_create(256, 256, 3, 1, 1, 4, 4, aqd.pack_codes(case.w_fields, 4), case.levels, wenc=1)
    rng = np.random.Generator(np.random.PCG64(94))
    try:
        segs, want = [], []
        for lv, (h, w) in enumerate(sizes):
            x = rng.integers(0, 16, size=(6, h, w, 256))
            y = torch.full((6, h, w, 128), 0xA5, dtype=torch.uint8, device="cuda:0")
            segs.append((handle, lv, 6, h, w, torch.from_numpy(aqd.pack_codes(x, 4)).cuda(), None, 0, 0, y))
            t = case.levels[lv]
            want.append(ref.pack_codes(ref.qconv(x, case.w_fields, 4, 1, 1, t["bias"], wenc=1, mult=t["mult"],
                                                 shift=t["shift"], bits_out=4), 4))
        aqd.qconv_run_group(segs)
        torch.cuda.synchronize()
        for s, w in zip(segs, want):
            assert_same(s[-1].cpu().numpy(), w, f"level of {s[3]} x {s[4]}")
    finally:
        aqd.qconv_destroy(handle)
