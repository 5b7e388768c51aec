// C-ABI host code: argument validation, handle creation (weight decoding and
// tiling, epilogue tables), kernel selection and launch, and the host-side
// parameter derivation helpers. Declarations and contracts: include/aqd.h.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <new>
#include <string>
#include <vector>

#include "aqd.h"
#include "internal.h"

using namespace aqd;

namespace {

thread_local std::string g_err;

aqd_status_t fail(aqd_status_t st, const std::string &msg)
{
    g_err = msg;
    return st;
}

#define REQUIRE(cond, msg)                            \
    do {                                              \
        if (!(cond))                                  \
            return fail(AQD_ERR_INVALID, (msg));      \
    } while (0)

// code widths; 3-bit codes (Tables 2 and 4 of the paper) are stored one per
// 4-bit container, so that every kernel reads them as 4-bit codes
bool code_bits(int b) { return b == 2 || b == 3 || b == 4 || b == 8; }
int stored_bits(int b) { return b == 3 ? 4 : b; }

bool aligned16(const void *p) { return ((uintptr_t)p & 15u) == 0; }

bool overlap(const void *a, size_t na, const void *b, size_t nb)
{
    uintptr_t a0 = (uintptr_t)a, b0 = (uintptr_t)b;
    return na && nb && a0 < b0 + nb && b0 < a0 + na;
}

// Positions of the 64 channels of one K step after the kernel's widening of
// packed codes (see qconv_mfma.hip): LDS byte p holds channel sigma(p);
// 8-bit codes are staged in channel order.
int widened_channel(int bits_in, int p)
{
    if (bits_in == 8)
        return p;
    if (bits_in == 4)
        return 8 * (p / 8) + 2 * (p % 4) + ((p / 4) % 2);
    return 16 * (p / 16) + 4 * (p % 4) + ((p / 4) % 4);  // bits_in == 2
}

// Channel (within a workgroup tile) of MFMA row rho: a wave slice has
// 4 * cpl_rows = 16 * MI rows; lane group g of accumulator tile i of slice w
// holds channel w * 16 * MI + cpl * g + 4i + e, where cpl = 4 * MI is the
// number of consecutive channels a lane owns per pixel.
int tile_row_channel(int rho, int cpl)
{
    const int slice = 4 * cpl;  // rows per wave slice
    int w = rho / slice, rr = rho % slice;
    int i = rr / 16, g = (rr % 16) / 4, e = rr % 4;
    return w * slice + cpl * g + 4 * i + e;
}

// Block-float kernels, 2-bit codes: position kappa of a chunk of channels holds
// channel fp4_channel(kappa). 32 packed 2-bit codes (channels 32c .. 32c+31) are
// spread into 16 bytes: word 0 = the even channels
// of the first 16, word 1 = their odd ones, words 2 and 3 the same for the
// second 16; nibble n of a word is its n-th channel.
int fp4_channel(int kappa)
{
    const int c = kappa / 32, wd = (kappa % 32) / 8, n = kappa % 8;
    return 32 * c + 16 * (wd >> 1) + 2 * n + (wd & 1);
}

// e2m1 nibble of a small integer (|v| <= 3: 0, 1, 2, 3 -> 0x0, 0x2, 0x4, 0x5;
// bit 3 = sign)
uint8_t e2m1_nibble(int v)
{
    static const uint8_t mag[4] = {0x0, 0x2, 0x4, 0x5};
    return (uint8_t)((v < 0 ? 0x8 : 0x0) | mag[v < 0 ? -v : v]);
}

// 16 nibbles of two words to 6-bit fields: the kernels' spread6 (mfma_common.h),
// whose channel order the weights therefore share
void host_spread6(uint32_t a, uint32_t b, uint32_t *d)
{
    const uint32_t t = a << 2, w = b << 2 | a >> 30;
    d[0] = (a & 0x0F00F00Fu) | (t & 0xC03C03C0u);
    d[1] = (b & 0xF00F00F0u) | (w & 0x03C03C03u);
    d[2] = (a & 0x00F00F00u) | (w & 0x3C03C03Cu);
}

// Weights of the global-fed kernel (internal.h): row r of row tile i of
// 64-channel group ct is channel 64 ct + 16 (r / 4) + 4 i + r % 4 (a lane then
// holds consecutive channels of its pixel); chunk g of K step ks is chunk
// 4 ks + g of the window, taps in order; chunks past the window are zeros.
// wv: decoded values [cout][taps][cin].
// packed: the same weights as 4-bit fields (else null), value: what a field decodes to.
std::vector<uint8_t> gf_weights(int kind, int cout, int taps, int cin, int groups, int steps, const int16_t *wv,
                                const uint8_t *packed, const int16_t *value)
{
    uint8_t mag[256], sgn[256];   // per byte of two fields: magnitudes, 2 where negative
    if (packed)
        for (int b = 0; b < 256; ++b) {
            const int lo = value[b & 15], hi = value[b >> 4];
            mag[b] = (uint8_t)((lo < 0 ? -lo : lo) | (hi < 0 ? -hi : hi) << 4);
            sgn[b] = (uint8_t)((lo < 0 ? 2 : 0) | (hi < 0 ? 32 : 0));
        }
    const int ch = kind == GF_I8 ? 16 : 32, chunks = taps * (cin / ch);
    const size_t tile = kind == GF_F6 ? GF_F6_TILE : 1024;
    std::vector<uint8_t> out((size_t)groups * steps * 4 * tile, 0);
    int order[32];
    for (int p = 0; p < ch; ++p)
        order[p] = kind == GF_F4 ? fp4_channel(p) : p;
    for (int co = 0; co < cout; ++co) {
        const int ct = co / 64, i = co % 16 / 4, r = 4 * (co % 64 / 16) + co % 4;
        // (the chunks of a channel's taps are consecutive: cin is a multiple of ch)
        for (int kc = 0; kc < chunks; ++kc) {
            const int16_t *src = wv + (size_t)co * taps * cin + (size_t)kc * ch;
            uint8_t *t = out.data() + (((size_t)ct * steps + kc / 4) * 4 + i) * tile;
            const int lane = 16 * (kc % 4) + r;
            if (kind == GF_F6) {
                // e2m3 of w / 8, |w| <= 15: sign and magnitude in 6-bit fields. The
                // magnitudes as packed nibbles go through the kernel's own widening,
                // and so do the signs, four bits up (bit 5 of a field = bit 1 of the
                // nibble)
                uint32_t w[6];
                for (int h = 0; h < 2; ++h) {
                    uint32_t m[2] = {0, 0}, sg[2] = {0, 0};
                    if (packed) {
                        const uint8_t *f = packed + ((size_t)co * taps * cin + (size_t)kc * ch + 16 * h) / 2;
                        for (int c = 0; c < 8; ++c) {
                            m[c / 4] |= (uint32_t)mag[f[c]] << (8 * (c % 4));
                            sg[c / 4] |= (uint32_t)sgn[f[c]] << (8 * (c % 4));
                        }
                    }
                    for (int c = 0; c < 16 && !packed; ++c) {
                        const int v = src[16 * h + c], neg = v < 0;
                        m[c / 8] |= (uint32_t)(neg ? -v : v) << (4 * (c % 8));
                        sg[c / 8] |= (uint32_t)(neg ? 2 : 0) << (4 * (c % 8));
                    }
                    uint32_t a[3], b[3];
                    host_spread6(m[0], m[1], a);
                    host_spread6(sg[0], sg[1], b);
                    w[3 * h] = a[0] | b[0] << 4;
                    w[3 * h + 1] = a[1] | b[1] << 4 | b[0] >> 28;
                    w[3 * h + 2] = a[2] | b[2] << 4 | b[1] >> 28;
                }
                std::memcpy(t + 16 * lane, w, 16);
                std::memcpy(t + 1024 + 8 * lane, w + 4, 8);
            } else if (kind == GF_F4) {
                for (int p = 0; p < 32; ++p)
                    t[16 * lane + p / 2] |= (uint8_t)(e2m1_nibble(src[order[p]]) << (4 * (p % 2)));
            } else {
                for (int p = 0; p < 16; ++p)
                    t[16 * lane + p] = (uint8_t)(int8_t)src[p];
            }
        }
    }
    return out;
}

// Requantisation in fp32 (Eq. 2 on integers, reading R2: code m and above from the
// accumulator T_m = ceil((2m - 1) 2^(d-1) / M) on, d = 31 + shift). floor(v a + b) in
// one fused multiply-add gives the same code for every integer v that fp32 holds
// (|v| <= 2^24) if
//     T_m a + b >= m   and   (T_m - 1) a + b <= m - ulp    for m = 1 .. qmax,
// since the rounded value is monotone in the exact one, m and the next smaller float
// are floats, and both sides are monotone in v. a = M / 2^d rounded to fp32, or a
// neighbour of it; *lo .. *hi is the interval that remains for b (usually a large
// part of a, always some of it but for the rounding of a). False if none does: the
// level then keeps the integer form.
bool float_requant(int mult, int shift, int qmax, float *a, double *lo, double *hi)
{
    if (mult <= 0 || shift < 2 || shift > 28)
        return false;
    const int d = 31 + shift;
    const float a0 = (float)std::ldexp((double)mult, -d);
    double t[16], width = -1.0;
    for (int m = 1; m <= qmax; ++m) {
        const uint64_t num = (uint64_t)(2 * m - 1) << (d - 1);   // < 2^5 * 2^58
        t[m] = (double)((num + (uint64_t)mult - 1) / (uint64_t)mult);
    }
    for (int step = 0; step <= 4 && width < 8e-6; ++step)
        for (int sign = -1; sign <= (step ? 1 : -1); sign += 2) {
            float c = a0;
            for (int k = 0; k < step; ++k)
                c = std::nextafterf(c, sign > 0 ? 2 * a0 : 0.f);
            double l = -1e30, u = 1e30;
            for (int m = 1; m <= qmax; ++m) {
                const double at = m - t[m] * c, below = m - m * 0x1p-23 - (t[m] - 1) * c;
                l = at > l ? at : l;
                u = below < u ? below : u;
            }
            if (u - l > width) {
                width = u - l;
                *a = c;
                *lo = l + 1e-9;   // (the doubles above are within 1e-13)
                *hi = u - 1e-9;
            }
        }
    return width > 2e-9;
}

// b for accumulators that lack `missing`: v = acc + missing
bool float_offset(float a, double lo, double hi, double missing, int32_t *bits)
{
    const double at = missing * a;
    const float b = (float)(at + (lo + hi) / 2);
    std::memcpy(bits, &b, 4);
    return b - at >= lo && b - at <= hi;
}

int pick_tile(int cout, bool codes, int bits_in)
{
    if (bits_in == 4 && cout >= 256 && (!codes || cout % 32 == 0))
        return TILE_256x128;
    return cout > 64 ? TILE_128x256 : TILE_64x512;
}

// 256 zero bytes per device: the source of the kernel's copies for padding taps.
std::mutex g_zero_mu;
void *g_zero[64] = {};

const uint8_t *device_zero_page()
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64)
        return nullptr;
    std::lock_guard<std::mutex> lock(g_zero_mu);
    if (!g_zero[dev]) {
        static const uint8_t zeros[256] = {};
        void *p = nullptr;
        if (hipMalloc(&p, sizeof zeros) != hipSuccess)
            return nullptr;
        if (hipMemcpy(p, zeros, sizeof zeros, hipMemcpyHostToDevice) != hipSuccess) {
            (void)hipFree(p);
            return nullptr;
        }
        g_zero[dev] = p;
    }
    return (const uint8_t *)g_zero[dev];
}

int weight_value(int field, int bits, int wenc)
{
    if (wenc == AQD_WENC_PAPER_ODD)
        return 2 * field - ((1 << bits) - 1);
    return field >= (1 << (bits - 1)) ? field - (1 << bits) : field;
}

}  // namespace

struct qconv_s {
    qconv_desc_t d;     // widths as stored (3-bit codes in 4-bit containers)
    int qmax;           // largest output code, 2^bits_out - 1 of the caller's bits_out
    bool mfma;
    int tile_cfg, blk_co, blk_px;
    int co_tiles, ksteps, cout_pad;
    void *w_dev;       // the one allocation: weights, then the parts below
    int32_t *epi_dev;  // [num_levels][EPI_FIELDS][cout_pad], and again for fp32 requantisation if a level has it
    int32_t *lut_dev;  // code skips: [num_levels][cout_pad][2^skip_bits] RSM(k, c, d), else null
    int32_t *lutf_dev, *gf_lutf;  // the same shape: fp32 b per code
    // per level: 1 = every shift >= 2, 2 = fp32 requantisation too; gf_fast: for the
    // block-float kernels, whose accumulators enter it without the bias
    std::vector<int> fast, gf_fast;
    std::vector<int> side0; // per level: every skip side is 0
    const uint8_t *zero;    // the device's zero page
    // global-fed kernel: operand kind (GF_NONE: not available), 64-channel
    // groups, K steps, weights and epilogue tables [num_levels][EPI_FIELDS][64 * gf_groups]
    int gf_kind, gf_groups, gf_steps;
    void *gf_w;
    int32_t *gf_epi;
};

extern "C" {

const char *aqd_last_error(void) { return g_err.c_str(); }

static aqd_status_t validate_desc(const qconv_desc_t *d)
{
    REQUIRE(d->cin >= 1 && d->cout >= 1, "cin and cout must be >= 1");
    REQUIRE(d->cin <= 65536 && d->cout <= 65536, "cin and cout must be <= 65536");
    REQUIRE(d->kh >= 1 && d->kh <= 7 && d->kw >= 1 && d->kw <= 7, "kh and kw must be in 1..7");
    REQUIRE(d->stride >= 1 && d->stride <= 4, "stride must be in 1..4");
    REQUIRE(d->pad >= 0 && d->pad < d->kh && d->pad < d->kw, "pad must be in 0..k-1");
    REQUIRE(code_bits(d->bits_in), "bits_in must be 2, 3, 4 or 8");
    REQUIRE(code_bits(d->bits_w), "bits_w must be 2, 3, 4 or 8");
    REQUIRE(d->wenc == AQD_WENC_TWOS || d->wenc == AQD_WENC_PAPER_ODD, "unknown weight grid");
    REQUIRE(d->out_mode == AQD_OUT_CODES || d->out_mode == AQD_OUT_INT32, "unknown output mode");
    REQUIRE((d->cin * stored_bits(d->bits_in)) % 8 == 0, "cin * bits_in must be a multiple of 8");
    REQUIRE((d->cin * stored_bits(d->bits_w)) % 8 == 0, "cin * bits_w must be a multiple of 8");
    if (d->out_mode == AQD_OUT_CODES) {
        REQUIRE(code_bits(d->bits_out), "bits_out must be 2, 3, 4 or 8");
        REQUIRE((d->cout * stored_bits(d->bits_out)) % 8 == 0, "cout * bits_out must be a multiple of 8");
    }
    REQUIRE(d->skip_bits == 0 || code_bits(d->skip_bits) || d->skip_bits == 32,
            "skip_bits must be 0, 2, 3, 4, 8 or 32");
    if (d->skip_bits) {
        REQUIRE(d->out_mode == AQD_OUT_CODES, "a skip add needs code output");
        REQUIRE((d->cout * stored_bits(d->skip_bits)) % 8 == 0, "cout * skip_bits must be a multiple of 8");
    }
    REQUIRE(d->skip_up2 == 0 || (d->skip_up2 == 1 && d->skip_bits), "skip_up2 needs a skip");
    REQUIRE(d->num_levels >= 1 && d->num_levels <= 64, "num_levels must be in 1..64");
    const double steps[3] = {d->step_in, d->step_w, d->step_out};
    for (double st : steps)
        REQUIRE(std::isfinite(st) && st >= 0.0, "step sizes must be finite and >= 0 (0: not given)");
    return AQD_OK;
}

aqd_status_t qconv_create(const qconv_desc_t *desc, const uint8_t *w_packed,
                          const qconv_epilogue_t *levels, qconv_t *out)
{
    REQUIRE(desc && w_packed && levels && out, "null argument");
    *out = nullptr;
    aqd_status_t st = validate_desc(desc);
    if (st != AQD_OK)
        return st;
    const qconv_desc_t dc = *desc;  // the caller's widths
    const bool codes = dc.out_mode == AQD_OUT_CODES;
    qconv_desc_t d = dc;             // stored widths
    d.bits_in = stored_bits(dc.bits_in);
    d.bits_w = stored_bits(dc.bits_w);
    if (codes)
        d.bits_out = stored_bits(dc.bits_out);
    if (dc.skip_bits && dc.skip_bits != 32)
        d.skip_bits = stored_bits(dc.skip_bits);
    for (int l = 0; l < d.num_levels; ++l) {
        const qconv_epilogue_t &e = levels[l];
        REQUIRE(e.bias, "epilogue bias is null");
        if (codes) {
            REQUIRE(e.mult && e.shift, "epilogue mult/shift is null");
            for (int c = 0; c < d.cout; ++c)
                REQUIRE(e.shift[c] >= -31 && e.shift[c] <= 31, "shift outside [-31, 31]");
        }
        if (d.skip_bits) {
            REQUIRE(e.skip_c && e.skip_d && e.skip_side, "skip parameters are null");
            for (int c = 0; c < d.cout; ++c) {
                REQUIRE(e.skip_d[c] >= 0 && e.skip_d[c] <= 31, "skip_d outside [0, 31]");
                REQUIRE(e.skip_side[c] == 0 || e.skip_side[c] == 1, "skip_side must be 0 or 1");
            }
        }
    }
    // accumulator bound: K * max code * max |weight| < 2^31
    const long long K = (long long)d.kh * d.kw * d.cin;
    const long long wmax = dc.wenc == AQD_WENC_PAPER_ODD ? (1 << dc.bits_w) - 1 : (1 << (dc.bits_w - 1));
    if (K * ((1 << dc.bits_in) - 1) * wmax >= (1LL << 31))
        return fail(AQD_ERR_UNSUPPORTED, "accumulator could exceed int32 for this K and bitwidths");

    // decode weight fields: value[] for everything a stored field can hold (a 3-bit
    // weight is the low three bits of its container, whatever the fourth is)
    int16_t value[256];
    for (int f = 0; f < (1 << d.bits_w); ++f)
        value[f] = (int16_t)weight_value(f & ((1 << dc.bits_w) - 1), dc.bits_w, d.wenc);
    const int per = 8 / d.bits_w;
    const int wrow = d.cin * d.bits_w / 8;
    const int taps = d.kh * d.kw;
    std::vector<int16_t> wv((size_t)d.cout * taps * d.cin);
    for (int co = 0; co < d.cout; ++co)
        for (int t = 0; t < taps; ++t) {
            const uint8_t *row = w_packed + ((size_t)co * taps + t) * wrow;
            int16_t *dst = wv.data() + ((size_t)co * taps + t) * d.cin;
            for (int b = 0; b < wrow; ++b)
                for (int e = 0; e < per; ++e)
                    dst[b * per + e] = value[(row[b] >> (e * d.bits_w)) & ((1 << d.bits_w) - 1)];
        }

    // MFMA kernel: 2/4-bit activations, weights that fit int8, 64-channel K
    // steps, output and skip codes of the input's width; the direct kernel
    // takes everything else
    const bool w_fits_i8 = dc.bits_w <= 4 || d.wenc == AQD_WENC_TWOS;
    // 8-bit codes with int32 outputs (the prediction convolutions of the
    // fully quantized networks): the int8 MFMA on codes re-centred by -128
    const bool b8 = dc.bits_in == 8 && !codes && d.skip_bits == 0 && d.cin % 128 == 0 && w_fits_i8 &&
                    d.cout % 4 == 0;
    // 4-bit codes in, 8-bit codes out (the last tower layer before 8-bit
    // prediction convolutions): the register-fed kernel's 8-bit epilogue
    const bool wv8 = d.bits_in == 4 && codes && dc.bits_out == 8 && d.skip_bits == 0 && d.cin % 256 == 0 &&
                     d.cout >= 256 && d.cout % 32 == 0 && w_fits_i8;
    // the ResNet stem (7x7, stride 2, pad 3) on a 3-channel 8-bit image
    const bool stem = dc.bits_in == 8 && d.cin == 3 && d.kh == 7 && d.kw == 7 && d.stride == 2 &&
                      d.pad == 3 && d.skip_bits == 0 && (!codes || dc.bits_out == 4) && d.cout % 64 == 0 &&
                      w_fits_i8;
    const bool mfma = b8 || wv8 || stem || ((d.bits_in == 2 || d.bits_in == 4) && d.cin % KC == 0 && w_fits_i8 &&
                             (codes ? (d.cout % 16 == 0 && d.bits_out == d.bits_in &&
                                       (d.skip_bits == 0 || d.skip_bits == d.bits_in || d.skip_bits == 32))
                                    : d.cout % 4 == 0));
    // 2-bit codes and weights in 256-channel chunks: block-float kernels only, exact
    // while every partial sum stays below 2^24 (K * 3 * max|w| < 2^24)
    const char *no_fp4 = std::getenv("AQD_NO_FP4");
    const bool fp4 = mfma && !(no_fp4 && std::strcmp(no_fp4, "1") == 0) && dc.bits_in == 2 && dc.bits_w == 2 &&
                     d.cin % 256 == 0 && d.cout % 256 == 0 &&
                     (codes ? (dc.bits_out == 2 && (d.skip_bits == 0 || d.skip_bits == 2)) : d.skip_bits == 0) &&
                     K * 3 * wmax < (1LL << 24);
    qconv_s h{};
    h.d = d;
    h.qmax = codes ? (1 << dc.bits_out) - 1 : 0;
    h.mfma = mfma;
    int cpl = 0;
    h.tile_cfg = fp4 ? TILE_FP4 : b8 ? TILE_B8 : stem ? TILE_STEM : pick_tile(d.cout, codes, d.bits_in);
    mfma_tile_shape(h.tile_cfg, &h.blk_co, &h.blk_px, &cpl);
    const int BLK_CO = h.blk_co;
    h.co_tiles = mfma ? (d.cout + BLK_CO - 1) / BLK_CO : 1;
    h.cout_pad = mfma ? h.co_tiles * BLK_CO : d.cout;
    h.ksteps = stem ? 4 : mfma ? taps * (d.cin / KC) : 0;
    h.fast.assign(d.num_levels, 0);
    h.gf_fast.assign(d.num_levels, 0);
    h.side0.assign(d.num_levels, 0);
    for (int l = 0; l < d.num_levels && d.skip_bits; ++l) {  // (stored widths from here on)
        int ok = 1;
        for (int c = 0; c < d.cout; ++c)
            ok &= levels[l].skip_side[c] == 0;
        h.side0[l] = ok;
    }
    for (int l = 0; l < d.num_levels && codes; ++l) {
        int ok = 1;
        for (int c = 0; c < d.cout; ++c)
            ok &= levels[l].shift[c] >= 2;
        h.fast[l] = ok;
    }

    std::vector<uint8_t> wbuf;
    if (stem) {
        // [co_tile][K step][row tile][lane][16 B], lane = 16 (16-byte column) + row:
        // K byte k = window row k / 32, tap k % 32 / 4, channel k % 4 (else zero);
        // channel tile_row_channel(rho) of the 64-channel tile
        wbuf.assign((size_t)h.co_tiles * 4 * 64 * KC, 0);
        for (int ct = 0; ct < h.co_tiles; ++ct)
            for (int rho = 0; rho < 64; ++rho) {
                const int co = ct * 64 + tile_row_channel(rho, cpl);
                for (int kh = 0; kh < 7; ++kh)
                    for (int kw = 0; kw < 7; ++kw)
                        for (int c = 0; c < 3; ++c) {
                            const int k = 32 * kh + 4 * kw + c;
                            const int lane = k % KC / 16 * 16 + rho % 16;
                            wbuf[((((size_t)ct * 4 + k / KC) * 4 + rho / 16) * 64 + lane) * 16 + k % 16] =
                                (uint8_t)(int8_t)wv[((size_t)co * taps + kh * 7 + kw) * d.cin + c];
                        }
            }
    } else if (fp4) {
        // (every launch runs on the block-float kernels, with weights of their own)
    } else if (mfma) {
        // tiles [co_tile][k step][row rho][byte p]: channel tile_row_channel(rho) of the tile,
        // input channel widened_channel(p) of the K step's 64-channel chunk
        const int kpt = d.cin / KC;
        int order[KC];
        for (int p = 0; p < KC; ++p)
            order[p] = widened_channel(d.bits_in, p);
        wbuf.assign((size_t)h.co_tiles * h.ksteps * BLK_CO * KC, 0);
        for (int ct = 0; ct < h.co_tiles; ++ct)
            for (int ks = 0; ks < h.ksteps; ++ks) {
                const int tap = ks / kpt, cc = ks % kpt;
                for (int rho = 0; rho < BLK_CO; ++rho) {
                    const int co = ct * BLK_CO + tile_row_channel(rho, cpl);
                    if (co >= d.cout)
                        continue;
                    int8_t *dst = (int8_t *)wbuf.data() + (((size_t)ct * h.ksteps + ks) * BLK_CO + rho) * KC;
                    const int16_t *src = wv.data() + ((size_t)co * taps + tap) * d.cin + cc * KC;
                    for (int p = 0; p < KC; ++p)
                        dst[p] = (int8_t)src[order[p]];
                }
            }
    } else {
        wbuf.resize(wv.size() * sizeof(int16_t));
        std::memcpy(wbuf.data(), wv.data(), wbuf.size());
    }
    // 8-bit codes on the MFMA enter as a - 128: the bias carries 128 * sum(w)
    // of the channel (every tap, padding included, enters as 0 - 128)
    std::vector<long long> recentre(d.cout, 0);
    if (b8 || stem)
        for (int co = 0; co < d.cout; ++co) {
            long long sw = 0;
            for (size_t k = 0; k < (size_t)taps * d.cin; ++k)
                sw += wv[(size_t)co * taps * d.cin + k];
            recentre[co] = 128 * sw;
        }
    std::vector<int32_t> epi((size_t)d.num_levels * EPI_FIELDS * h.cout_pad, 0);
    for (int l = 0; l < d.num_levels; ++l) {
        const qconv_epilogue_t &e = levels[l];
        int32_t *t = epi.data() + (size_t)l * EPI_FIELDS * h.cout_pad;
        for (int c = 0; c < d.cout; ++c) {
            const long long b = (long long)e.bias[c] + recentre[c];
            if (b < INT32_MIN || b > INT32_MAX)
                return fail(AQD_ERR_UNSUPPORTED, "bias + 128 * sum(w) exceeds int32 (8-bit codes)");
            t[EPI_BIAS * h.cout_pad + c] = (int32_t)b;
            if (codes) {
                const int sh = e.shift[c];
                t[EPI_MULT * h.cout_pad + c] = e.mult[c];
                t[EPI_SHIFT * h.cout_pad + c] = sh;
                t[EPI_SHR * h.cout_pad + c] = sh - 1;
                t[EPI_RND * h.cout_pad + c] = sh >= 2 ? 1 << (sh - 2) : 0;
            }
            if (d.skip_bits) {
                t[EPI_SKIP_C * h.cout_pad + c] = e.skip_c[c];
                t[EPI_SKIP_D * h.cout_pad + c] = e.skip_d[c];
                t[EPI_SKIP_SIDE * h.cout_pad + c] = e.skip_side[c];
            }
        }
    }

    // code skips: per level and channel the skip operand's scaled value
    // RSM(k, c, d) for every code k (used when every side of the level is 0),
    // computed exactly and kept modulo 2^32 as the kernels' 32-bit sums are
    std::vector<int32_t> lut;
    const int nk = (d.skip_bits > 0 && d.skip_bits < 32) ? (1 << d.skip_bits) : 0;
    if (nk) {
        lut.assign((size_t)d.num_levels * h.cout_pad * nk, 0);
        for (int l = 0; l < d.num_levels; ++l)
            for (int c = 0; c < d.cout; ++c) {
                const long long cc = levels[l].skip_c[c];
                const int dd = levels[l].skip_d[c];
                for (int k = 0; k < nk; ++k) {
                    const long long p = (long long)k * cc;
                    const long long r = dd > 0 ? (p + (1LL << (dd - 1))) >> dd : p;
                    lut[((size_t)l * h.cout_pad + c) * nk + k] = (int32_t)(uint32_t)(uint64_t)r;
                }
            }
    }

    // the global-fed kernel: 4-bit containers with weights of at most 4 bits and
    // 2-bit codes with 2-bit weights while every sum stays exact in fp32, 8-bit
    // codes with int8 weights while the re-centred bias fits int32
    std::vector<uint8_t> gfw;
    std::vector<int32_t> gfe;
    if (!codes || d.cout % 4 == 0) {
        const long long kmax = K * ((1 << dc.bits_in) - 1) * wmax;
        const bool off2 = no_fp4 && std::strcmp(no_fp4, "1") == 0;   // 2-bit layers on int8
        if (dc.bits_in >= 3 && dc.bits_in <= 4 && dc.bits_w <= 4 && d.cin % 32 == 0 && kmax < (1LL << 24))
            h.gf_kind = GF_F6;
        else if (!off2 && dc.bits_in == 2 && dc.bits_w == 2 && d.cin % 32 == 0 && kmax < (1LL << 24))
            h.gf_kind = GF_F4;
        else if (dc.bits_in == 8 && d.cin % 16 == 0 && w_fits_i8)
            h.gf_kind = GF_I8;
    }
    if (h.gf_kind != GF_NONE) {
        const int chunk = h.gf_kind == GF_I8 ? 16 : 32;
        h.gf_groups = (d.cout + 63) / 64;
        h.gf_steps = (taps * (d.cin / chunk) + 3) / 4;
        gfw = gf_weights(h.gf_kind, d.cout, taps, d.cin, h.gf_groups, h.gf_steps, wv.data(),
                         d.bits_w == 4 ? w_packed : nullptr, value);
        const int pad = 64 * h.gf_groups;
        gfe.assign((size_t)d.num_levels * EPI_FIELDS * pad, 0);
        for (int l = 0; l < d.num_levels && h.gf_kind != GF_NONE; ++l)
            for (int f = 0; f < EPI_FIELDS; ++f)
                std::memcpy(gfe.data() + ((size_t)l * EPI_FIELDS + f) * pad,
                            epi.data() + ((size_t)l * EPI_FIELDS + f) * h.cout_pad, d.cout * sizeof(int32_t));
        if (h.gf_kind == GF_I8 && !b8)   // (b8 tables are re-centred already)
            for (int l = 0; l < d.num_levels; ++l)
                for (int co = 0; co < d.cout; ++co) {
                    long long sw = 0;
                    for (size_t k = 0; k < (size_t)taps * d.cin; ++k)
                        sw += wv[(size_t)co * taps * d.cin + k];
                    const long long b = (long long)levels[l].bias[co] + 128 * sw;
                    if (b < INT32_MIN || b > INT32_MAX)
                        h.gf_kind = GF_NONE;   // runs on the direct kernel
                    gfe[((size_t)l * EPI_FIELDS + EPI_BIAS) * pad + co] = (int32_t)b;
                }
    }

    // fp32 requantisation, where it is exact: codes of at most 4 bits, no skip or code
    // skips of side 0 (an offset per code). a and b per channel, for v = acc + bias
    // (tables and lutf; the stem's for v = acc) and for the block-float accumulators (gf tables and glutf)
    std::vector<int32_t> lutf(lut.size()), glutf(lut.size());
    std::vector<int32_t> epif(epi);   // the same tables with a and b
    const int qmax = codes ? (1 << dc.bits_out) - 1 : 0;
    for (int l = 0; l < d.num_levels && codes && dc.bits_out <= 4 && d.skip_bits <= 4; ++l) {
        if (!h.fast[l] || (d.skip_bits && !h.side0[l]))
            continue;
        const qconv_epilogue_t &e = levels[l];
        int32_t *t = epif.data() + (size_t)l * EPI_FIELDS * h.cout_pad;
        const int gpad = 64 * h.gf_groups;
        int32_t *gt = gfe.data() + (size_t)l * EPI_FIELDS * gpad;
        const float unit = h.gf_kind == GF_F6 ? 64.f : h.gf_kind == GF_F4 ? 2.f : 1.f;
        bool ok = true, gok = h.gf_kind != GF_NONE;
        for (int c = 0; c < d.cout && (ok || gok); ++c) {
            float a = 0.f;
            double lo = 0, hi = 0;
            if (!float_requant(e.mult[c], e.shift[c], qmax, &a, &lo, &hi)) {
                ok = gok = false;
                break;
            }
            // (the tables' bias: re-centred for 8-bit codes)
            const double bias = t[EPI_BIAS * h.cout_pad + c];
            ok = ok && K * ((1 << dc.bits_in) - 1) * wmax + std::fabs(bias) < (1 << 24);
            std::memcpy(&t[EPI_FA * h.cout_pad + c], &a, 4);
            ok = ok && float_offset(a, lo, hi, stem ? bias : 0, &t[EPI_FB * h.cout_pad + c]);
            if (gok) {
                const double gbias = gt[EPI_BIAS * gpad + c];
                const float ga = a * unit;
                std::memcpy(&gt[EPI_FA * gpad + c], &ga, 4);
                gok = h.gf_kind != GF_I8 || K * ((1 << dc.bits_in) - 1) * wmax < (1 << 24);
                gok = gok && float_offset(a, lo, hi, gbias, &gt[EPI_FB * gpad + c]);
            }
            for (int k = 0; k < nk; ++k) {
                const size_t at = ((size_t)l * h.cout_pad + c) * nk + k;
                const long long p = (long long)k * e.skip_c[c];
                const int dd = e.skip_d[c];
                const double r = (double)(dd > 0 ? (p + (1LL << (dd - 1))) >> dd : p);
                ok = ok && float_offset(a, lo, hi, r, &lutf[at]);
                gok = gok && float_offset(a, lo, hi, r + gt[EPI_BIAS * gpad + c], &glutf[at]);
            }
        }
        if (ok)
            h.fast[l] = 2;
        if (gok)
            h.gf_fast[l] = 2;
    }
    for (int l = 0; l < d.num_levels; ++l)
        if (!h.gf_fast[l])
            h.gf_fast[l] = h.fast[l] ? 1 : 0;
    if (std::count(h.fast.begin(), h.fast.end(), 2))
        epi.insert(epi.end(), epif.begin(), epif.end());

    const char *inject = std::getenv("AQD_FAULT_INJECT");
    if (inject && std::strcmp(inject, "alloc") == 0)
        return fail(AQD_ERR_NOMEM, "device allocation failed (injected)");

    h.zero = device_zero_page();
    if (!h.zero)
        return fail(AQD_ERR_NOMEM, "could not allocate the device zero page");
    qconv_s *hp = new (std::nothrow) qconv_s(h);
    if (!hp)
        return fail(AQD_ERR_NOMEM, "host allocation failed");
    // one device allocation for the weights, the tables and the skip tables
    // (256-byte aligned parts). MFMA weights: four K steps of 256-row tiles
    // (64 KiB) of padding past the end, which the register-fed kernel's
    // look-ahead may read (never use)
    auto up = [](size_t b) { return (b + 255) & ~(size_t)255; };
    const size_t o_epi = up(wbuf.size() + (mfma && !fp4 ? 4 * 256 * KC : 0)), o_lut = o_epi + up(epi.size() * sizeof(int32_t)),
                 o_lutf = o_lut + up(lut.size() * sizeof(int32_t)), o_glutf = o_lutf + up(lut.size() * sizeof(int32_t)),
                 o_gfw = o_glutf + up(lut.size() * sizeof(int32_t)), o_gfe = o_gfw + up(gfw.size()),
                 total = o_gfe + gfe.size() * sizeof(int32_t);
    if (hipMalloc(&hp->w_dev, total) != hipSuccess) {
        delete hp;
        return fail(AQD_ERR_NOMEM, "hipMalloc of the weights and tables failed");
    }
    struct Part {
        size_t at;
        const void *src;
        size_t n;
    };
    const Part parts[7] = {{0, wbuf.data(), wbuf.size()},
                           {o_epi, epi.data(), epi.size() * sizeof(int32_t)},
                           {o_lut, lut.data(), lut.size() * sizeof(int32_t)},
                           {o_lutf, lutf.data(), lutf.size() * sizeof(int32_t)},
                           {o_glutf, glutf.data(), glutf.size() * sizeof(int32_t)},
                           {o_gfw, gfw.data(), gfw.size()},
                           {o_gfe, gfe.data(), gfe.size() * sizeof(int32_t)}};
    bool copied = true;
    if (total <= (256u << 10)) {   // small: one copy
        std::vector<uint8_t> blob(total, 0);
        for (const Part &q : parts)
            if (q.n)
                std::memcpy(blob.data() + q.at, q.src, q.n);
        copied = hipMemcpy(hp->w_dev, blob.data(), total, hipMemcpyHostToDevice) == hipSuccess;
    } else {
        for (const Part &q : parts)
            copied = copied && (!q.n || hipMemcpy((uint8_t *)hp->w_dev + q.at, q.src, q.n, hipMemcpyHostToDevice) ==
                                            hipSuccess);
    }
    if (!copied) {
        (void)hipFree(hp->w_dev);
        delete hp;
        return fail(AQD_ERR_DEVICE, "copy of the weights to the device failed");
    }
    uint8_t *base = (uint8_t *)hp->w_dev;
    hp->epi_dev = (int32_t *)(base + o_epi);
    hp->lut_dev = nk ? (int32_t *)(base + o_lut) : nullptr;
    hp->lutf_dev = nk ? (int32_t *)(base + o_lutf) : nullptr;
    hp->gf_lutf = nk ? (int32_t *)(base + o_glutf) : nullptr;
    hp->gf_w = base + o_gfw;
    hp->gf_epi = (int32_t *)(base + o_gfe);
    *out = hp;
    return AQD_OK;
}

const char *qconv_path(qconv_t conv)
{
    if (!conv)
        return "invalid";
    if (!conv->mfma)
        return "direct";
    return conv->tile_cfg == TILE_FP4 ? "fp4-mfma" : "i8-mfma";  // TILE_B8 included
}

void qconv_destroy(qconv_t conv)
{
    if (!conv)
        return;
    (void)hipFree(conv->w_dev);
    delete conv;
}

aqd_status_t qconv_out_shape(qconv_t conv, int h, int w, int *ho, int *wo)
{
    REQUIRE(conv && ho && wo, "null argument");
    REQUIRE(h >= 1 && w >= 1, "h and w must be >= 1");
    const qconv_desc_t &d = conv->d;
    REQUIRE(h + 2 * d.pad >= d.kh && w + 2 * d.pad >= d.kw, "input smaller than the filter");
    *ho = (h + 2 * d.pad - d.kh) / d.stride + 1;
    *wo = (w + 2 * d.pad - d.kw) / d.stride + 1;
    return AQD_OK;
}

aqd_status_t qconv_scales(qconv_t conv, double *alpha_conv, double *step_out)
{
    REQUIRE(conv, "null handle");
    REQUIRE(conv->d.step_in > 0.0 && conv->d.step_w > 0.0,
            "the handle was created without step_in / step_w");
    if (alpha_conv)
        *alpha_conv = conv->d.step_in * conv->d.step_w;
    if (step_out)
        *step_out = conv->d.step_out;
    return AQD_OK;
}

}  // extern "C"

namespace {

struct SegCheck {
    int ho, wo;
    size_t xbytes, sbytes, ybytes;
};

aqd_status_t check_seg(const qconv_seg_t &s, SegCheck *out)
{
    REQUIRE(s.conv, "null handle");
    const qconv_desc_t &d = s.conv->d;
    REQUIRE(s.level >= 0 && s.level < d.num_levels, "level out of range");
    REQUIRE(s.n >= 0, "n must be >= 0");
    int ho = 0, wo = 0;
    aqd_status_t st = qconv_out_shape(s.conv, s.h, s.w, &ho, &wo);
    if (st != AQD_OK)
        return st;
    REQUIRE((long long)s.n * ho * wo < (1LL << 31) && (long long)s.n * s.h * s.w < (1LL << 31),
            "too many pixels for one call");
    out->ho = ho;
    out->wo = wo;
    out->xbytes = (size_t)s.n * s.h * s.w * d.cin * d.bits_in / 8;
    out->ybytes = (size_t)s.n * ho * wo * d.cout * (d.out_mode == AQD_OUT_INT32 ? 32 : d.bits_out) / 8;
    out->sbytes = 0;
    if (s.n == 0)
        return AQD_OK;
    REQUIRE(s.x && s.y, "null tensor");
    REQUIRE(aligned16(s.x) && aligned16(s.y), "tensors must be 16-byte aligned");
    if (d.skip_bits) {
        REQUIRE(s.skip, "the handle has a skip but skip is null");
        REQUIRE(aligned16(s.skip), "skip must be 16-byte aligned");
        if (d.skip_up2)
            REQUIRE((ho - 1) / 2 < s.hs && (wo - 1) / 2 < s.ws && s.hs >= 1 && s.ws >= 1,
                    "upsampled skip too small for the output");
        else
            REQUIRE(s.hs == ho && s.ws == wo, "skip size must equal the output size");
        out->sbytes = (size_t)s.n * s.hs * s.ws * d.cout * d.skip_bits / 8;
    } else {
        REQUIRE(!s.skip, "skip given to a handle without a skip");
    }
    REQUIRE(!overlap(s.y, out->ybytes, s.x, out->xbytes), "output overlaps the input");
    REQUIRE(!overlap(s.y, out->ybytes, s.skip, out->sbytes), "output overlaps the skip");
    return AQD_OK;
}

bool same_config(const qconv_desc_t &a, const qconv_desc_t &b)
{
    return a.cin == b.cin && a.cout == b.cout && a.kh == b.kh && a.kw == b.kw &&
           a.stride == b.stride && a.pad == b.pad && a.bits_in == b.bits_in &&
           a.bits_w == b.bits_w && a.wenc == b.wenc && a.out_mode == b.out_mode &&
           (a.out_mode == AQD_OUT_INT32 || a.bits_out == b.bits_out) &&
           a.skip_bits == b.skip_bits && a.skip_up2 == b.skip_up2;
}

aqd_status_t launch_direct(const qconv_seg_t &s, const SegCheck &c, hipStream_t stream)
{
    const qconv_s &h = *s.conv;
    DirectArgs a{};
    a.x = (const uint8_t *)s.x;
    a.skip = s.skip;
    a.y = s.y;
    a.wt = (const int16_t *)h.w_dev;
    a.epi = h.epi_dev + (size_t)s.level * EPI_FIELDS * h.cout_pad;
    a.n = s.n;
    a.h = s.h;
    a.w = s.w;
    a.ho = c.ho;
    a.wo = c.wo;
    a.hs = s.hs;
    a.ws = s.ws;
    a.cin = h.d.cin;
    a.cout = h.d.cout;
    a.kh = h.d.kh;
    a.kw = h.d.kw;
    a.stride = h.d.stride;
    a.pad = h.d.pad;
    a.bits_in = h.d.bits_in;
    a.out_bits = h.d.out_mode == AQD_OUT_INT32 ? 32 : h.d.bits_out;
    a.qmax = h.qmax;
    a.skip_bits = h.d.skip_bits;
    a.up2 = h.d.skip_up2;
    if (launch_qconv_direct(a, stream) != hipSuccess)
        return fail(AQD_ERR_DEVICE, "direct conv launch failed");
    return AQD_OK;
}

}  // namespace

namespace {

// Checks a group and fills the MFMA launch description (everything but the
// split); *tiles receives the number of output tiles, *direct whether the
// group runs on the direct kernel.
aqd_status_t prepare_group(int count, const qconv_seg_t *segs, SegCheck *chk, MfmaArgs *out,
                           bool *direct)
{
    REQUIRE(segs && count >= 1 && count <= AQD_MAX_SEGS, "count must be in 1..AQD_MAX_SEGS");
    for (int i = 0; i < count; ++i) {
        aqd_status_t st = check_seg(segs[i], &chk[i]);
        if (st != AQD_OK)
            return st;
        // (the tile differs where handles were created with and without AQD_NO_FP4)
        REQUIRE(same_config(segs[0].conv->d, segs[i].conv->d) && segs[0].conv->qmax == segs[i].conv->qmax &&
                    segs[0].conv->tile_cfg == segs[i].conv->tile_cfg,
                "grouped handles must share shapes, bitwidths and modes");
    }
    for (int i = 0; i < count; ++i)
        for (int j = 0; j < count; ++j) {
            if (i == j || segs[j].n == 0 || segs[i].n == 0)
                continue;
            REQUIRE(!overlap(segs[i].y, chk[i].ybytes, segs[j].y, chk[j].ybytes) &&
                        !overlap(segs[i].y, chk[i].ybytes, segs[j].x, chk[j].xbytes) &&
                        !overlap(segs[i].y, chk[i].ybytes, segs[j].skip, chk[j].sbytes),
                    "a segment output overlaps another segment's tensors");
        }
    const qconv_s &h0 = *segs[0].conv;
    *direct = !h0.mfma;
    if (!h0.mfma)
        return AQD_OK;
    MfmaArgs &a = *out;
    a = MfmaArgs{};
    // launch tile for a handle laid out for 256-channel tiles: 1x1 convolutions
    // with cin <= 128 and code outputs on persistent 256 x 64 tiles (weights kept
    // in LDS, next tile's copies during the current epilogue); other short K
    // ranges with code outputs on 256 x 64 tiles three to a CU; launches with fewer
    // 256 x 128 tiles than CUs (but not tiny, and not so long in K that
    // splitting K is the better cure) on 256 x 64 tiles two to a CU (measured:
    // from ~260 tiles on, the larger tile is faster)
    int tile_cfg = h0.tile_cfg, blk_px = h0.blk_px;
    // the register-fed, block-float and 8-bit kernels address each segment's input
    // with 32-bit buffer offsets
    bool x_small = true;
    for (int i = 0; i < count; ++i)
        x_small = x_small && chk[i].xbytes < (1ull << 31);
    REQUIRE(x_small || (tile_cfg != TILE_FP4 && tile_cfg != TILE_B8),
            "2-bit (FP4) and 8-bit MFMA layers take inputs of less than 2^31 bytes per segment");
    long long t_handle = 0;  // tiles at the handle's own tile shape
    for (int i = 0; i < count; ++i)
        t_handle += ((long long)segs[i].n * chk[i].ho * chk[i].wo + h0.blk_px - 1) / h0.blk_px * h0.co_tiles;
    if (h0.tile_cfg == TILE_256x128) {
        long long t128 = 0;
        for (int i = 0; i < count; ++i)
            t128 += ((long long)segs[i].n * chk[i].ho * chk[i].wo + 127) / 128 * h0.co_tiles;
        const bool short_codes = h0.ksteps <= 4 && h0.d.out_mode == AQD_OUT_CODES && h0.d.bits_in == 4 &&
                                 h0.d.bits_out == 4 && (h0.d.skip_bits == 0 || h0.d.skip_bits == 4);
        // 1x1 layers with 256 input channels and 4-bit code outputs (one
        // segment): weight-stationary persistent tiles
        const bool wvs = count == 1 && h0.d.out_mode == AQD_OUT_CODES && h0.d.bits_in == 4 &&
                         h0.d.bits_out == 4 && (h0.d.skip_bits == 0 || h0.d.skip_bits == 4) && h0.d.kh == 1 &&
                         h0.d.kw == 1 && h0.d.pad == 0 && h0.d.cin == 256 &&
                         h0.d.cout % 256 == 0 && h0.co_tiles <= 256 && x_small;
        if (h0.d.out_mode == AQD_OUT_CODES && h0.d.bits_out == 8) {
            // 8-bit code outputs: only the register-fed kernel writes them
            REQUIRE(x_small, "8-bit code outputs take inputs of less than 2^31 bytes per segment");
            tile_cfg = TILE_WV;
        } else if (wvs) {
            tile_cfg = TILE_WVS;
            blk_px = 64;
        } else if (short_codes && h0.ksteps <= 2 && h0.d.kh == 1 && h0.d.kw == 1 && h0.d.pad == 0 &&
                   h0.d.cout % 256 == 0) {
            tile_cfg = TILE_STREAM;
            blk_px = 64;
        } else if (short_codes && h0.d.kh == 1 && h0.d.kw == 1 && h0.d.pad == 0 && h0.d.cout % 256 == 0 &&
                   h0.co_tiles <= 128) {
            // 3-4 K steps: the weights of a 256-row tile do not fit twice in
            // LDS, its 128-row halves do (persistent 128 x 64 tiles; the
            // streaming launch takes at most 256 channel tiles)
            tile_cfg = TILE_STREAM_H128;
            blk_px = 64;
        } else if (short_codes) {
            tile_cfg = TILE_256x64S;
            blk_px = 64;
        } else if (t128 >= 64 && t128 < 200 && h0.ksteps <= 80 && h0.d.bits_in == 4 && h0.d.cin % 256 == 0 &&
                   h0.d.out_mode == AQD_OUT_CODES && (h0.d.skip_bits == 0 || h0.d.skip_bits == 4) && x_small) {
            // fewer 256 x 128 tiles than CUs, 256-channel input chunks, code
            // outputs: register-fed 256 x 64 tiles, one round at three per CU
            // (longer K ranges split K instead)
            tile_cfg = TILE_WV64;
            blk_px = 64;
        } else if (t128 >= 64 && t128 < 200 && h0.ksteps <= 80) {
            tile_cfg = TILE_256x64;
            blk_px = 64;
        } else if (h0.d.bits_in == 4 && h0.d.cin % 256 == 0 &&
                   (h0.d.out_mode == AQD_OUT_CODES ? (h0.d.skip_bits == 0 || h0.d.skip_bits == 4)
                                                   : h0.d.skip_bits == 0) &&
                   t128 >= 200 && x_small) {
            // 256-channel input chunks: weights read into registers (no LDS
            // traffic for them), activation codes staged in LDS four K steps
            // at a time
            tile_cfg = TILE_WV;
        }
    } else if ((h0.tile_cfg == TILE_128x256 || h0.tile_cfg == TILE_64x512) && h0.ksteps <= 4 &&
               h0.d.out_mode == AQD_OUT_CODES && h0.d.bits_in == 4 && h0.d.bits_out == 4 &&
               h0.d.skip_bits == 0 && h0.d.kh == 1 && h0.d.kw == 1 && h0.d.pad == 0 &&
               h0.d.cout % h0.blk_co == 0 && h0.co_tiles <= 256) {
        // 1x1 convolutions with cin <= 256 on 128- or 64-channel handles:
        // persistent streaming tiles (weights resident in LDS)
        tile_cfg = h0.tile_cfg == TILE_128x256 ? TILE_STREAM_C128 : TILE_STREAM_C64;
        blk_px = h0.tile_cfg == TILE_128x256 ? 64 : 128;
    } else if ((h0.tile_cfg == TILE_128x256 || h0.tile_cfg == TILE_64x512) && t_handle > 256 && h0.d.bits_in == 4 &&
               h0.d.skip_bits == 0 && (h0.d.out_mode == AQD_OUT_INT32 || h0.d.bits_out == 4)) {
        tile_cfg = h0.tile_cfg == TILE_128x256 ? TILE_128x128_O3 : TILE_64x256_O3;
        blk_px = h0.tile_cfg == TILE_128x256 ? 128 : 256;
    }
    if (tile_cfg == TILE_WV && h0.d.out_mode == AQD_OUT_CODES) {
        // a little above one round of 256 x 128 tiles at one workgroup per CU
        // (the CUs that get a second tile set the launch's time): 256 x 144
        // tiles, one round
        long long t128 = 0, t144 = 0;
        for (int i = 0; i < count; ++i) {
            const long long p = (long long)segs[i].n * chk[i].ho * chk[i].wo;
            t128 += (p + 127) / 128 * h0.co_tiles;
            t144 += (p + 143) / 144 * h0.co_tiles;
        }
        if (h0.ksteps <= 8) {
            // short K ranges: a tile's copies and epilogue outweigh its MFMAs;
            // 256 x 64 tiles, three workgroups per CU
            tile_cfg = TILE_WV64;
            blk_px = 64;
        } else if (t128 > 256 && t144 <= 256) {
            tile_cfg = TILE_WV144;
            blk_px = 144;
        }
    }
    // the half view splits each 256-channel tile in two
    const int co_tiles = tile_cfg == TILE_STREAM_H128 ? 2 * h0.co_tiles : h0.co_tiles;
    int tiles = 0;
    for (int i = 0; i < count; ++i) {
        const qconv_seg_t &s = segs[i];
        if (s.n == 0)
            continue;
        MfmaSeg &m = a.seg[a.nseg++];
        m.x = (const uint8_t *)s.x;
        m.skip = s.skip;
        m.y = s.y;
        m.wt = (const int8_t *)s.conv->w_dev;
        m.epi = s.conv->epi_dev + (size_t)s.level * EPI_FIELDS * s.conv->cout_pad;
        m.P = (long long)s.n * chk[i].ho * chk[i].wo;
        m.n = s.n;
        m.h = s.h;
        m.w = s.w;
        m.ho = chk[i].ho;
        m.wo = chk[i].wo;
        m.hs = s.hs;
        m.ws = s.ws;
        m.tile_begin = tiles;
        m.fast = s.conv->fast[s.level];
        m.side0 = s.conv->side0[s.level];
        m.lut = s.conv->lut_dev ? s.conv->lut_dev + (size_t)s.level * s.conv->cout_pad * (1 << h0.d.skip_bits)
                                : nullptr;
        // (the stem's tiles lie in one image each, and its grid does not grow with them)
        const bool stem = tile_cfg == TILE_STEM;
        const long long px_tiles = stem ? (long long)m.n * ((m.ho + STEM_TH - 1) / STEM_TH) * ((m.wo + STEM_TW - 1) / STEM_TW)
                                        : (m.P + blk_px - 1) / blk_px;
        REQUIRE(tiles + px_tiles * co_tiles < (1LL << (stem ? 30 : 26)), "too many tiles for one launch");
        tiles += (int)(px_tiles * co_tiles);
    }
    // fp32 requantisation when every segment has it (4-bit codes in and out, the stem)
    bool f32 = (h0.d.bits_in == 4 || tile_cfg == TILE_STEM) && h0.d.out_mode == AQD_OUT_CODES && h0.d.bits_out == 4 && h0.d.skip_bits <= 4;
    for (int i = 0; i < a.nseg; ++i)
        f32 = f32 && a.seg[i].fast == 2;
    const size_t lut_words = (size_t)h0.cout_pad * (1 << (h0.d.skip_bits & 15));
    for (int i = 0, k = 0; i < count; ++i) {
        if (segs[i].n == 0)
            continue;
        MfmaSeg &m = a.seg[k++];
        if (!f32) {
            m.fast = m.fast ? 1 : 0;
            continue;
        }
        m.epi += (size_t)segs[i].conv->d.num_levels * EPI_FIELDS * h0.cout_pad;
        if (h0.d.skip_bits)
            m.lut = segs[i].conv->lutf_dev + segs[i].level * lut_words;
    }
    a.total_tiles = tiles;
    a.tiles_per_xcd = (tiles + 7) / 8;
    a.ksplit = 1;
    a.kchunk = h0.ksteps;
    a.part = 0;
    a.cin = h0.d.cin;
    a.cout = h0.d.cout;
    a.cout_pad = h0.cout_pad;
    a.kh = h0.d.kh;
    a.kw = h0.d.kw;
    a.stride = h0.d.stride;
    a.pad = h0.d.pad;
    a.co_tiles = co_tiles;
    a.ksteps = h0.ksteps;
    a.up2 = h0.d.skip_up2;
    a.tile_cfg = tile_cfg;
    a.bits_out = h0.d.out_mode == AQD_OUT_INT32 ? 32 : h0.d.bits_out;
    a.qmax = h0.qmax;
    a.skip_bits = h0.d.skip_bits;
    a.zero = h0.zero;
    return AQD_OK;
}

// The launch of a checked group on the block-float kernels (global-fed: qconv_gf,
// tiled: qconv_fx), if they are the better choice over the handles' own kernel
// (own: its tile, -1: the direct kernel). t64 counts tiles of 64 x 64 outputs,
// steps K steps of 128 channels (64 of 8-bit codes). Measured on MI355X, us per
// launch in a graph of 20, own -> new (P pixels; "gf n" n waves, "fx a x b" tiles):
//  * 3x3, stride 1, 64, 128 or a multiple of 256 channels in: fx3 from t64 200 on, 512 with
//    256 channels or more (256 -> 256 P 4200, t64 264: fx3 10.3, gf 11.3 on weights in the
//    L2, but in a network, where they are not, 15 and 12; 512 -> 512 P 1050: 16.0 and 10.6).
//    64 -> 64 P 534400 37.7 -> 27.1; 128 -> 128 P 133600 31.2 -> 21.2, with a skip 42.7 ->
//    26.0; 256 -> 256 P 33600 23.0 -> 20.6, P 133600 78 -> 55, P 267200 139 -> 94; 256 ->
//    720 int32 P 133600 235 -> 164; 512 -> 512 P 8400 39.7 -> 24.7. At 256 channels in and
//    up to 64 out gf stays up to t64 1100 (256 -> 36 P 66800: 23.1, fx3 26.1). 256 x 128
//    tiles where the tiles still fill the chip (P 16700: 14.3, 256 x 64 15.5; 256 -> 720 P
//    4200: 17.4, 13.0), at 2 bits 128 x 128 up to larger sizes (P 133600: 44.2, 42.0). Not
//    for more than 256 channels in and up to 128 out, where its 256 x 64 tiles are half
//    or more padding (3x3 512 -> 64 t64 8775: fx3 403 us, own 226; 512 -> 128 t64 13000:
//    fx3 261, fx 128 x 128 169, own 223), nor where the rows and columns of padding,
//    which fx3 computes like any pixel, make it slower than what follows: at (h + 1)
//    (w + 1) / (h w) = 1 it takes 0.60 of own's time at 256 -> 256 and t64 5000 (fx 0.75),
//    0.70 at 512 -> 512 and t64 2000 (fx 0.73), 0.86 at 256 -> 64 and 3000 (own 1), 0.5
//    at 128 -> 128 (own 1) and 0.33 at 64 -> 64 and 512 (gf 0.50); 512 -> 64 on images of
//    2 x 1 took 5.5 times own's;
//  * else t64 <= 512 (two tiles per CU): gf. 3x3 256 -> 256 P 4200 27.6 -> 11.3; 1x1 2048
//    -> 512 P 1050 21 -> 7.4; 3x3 stride 2 2048 -> 256 P 273 30 -> 21, P 2184 37 -> 29;
//    3x3 64 -> 64 P 1024 14.9 -> 4.6. So do the shapes of the direct kernel, at any
//    size (3x3 256 -> 1 P 44600 1470 -> 8). Code outputs of 1x1 layers of 4 bits and up
//    to 256 channels on the persistent tiles: gf over own 1.25 for 64 -> 64, 1.15 for 128
//    -> 64, 0.95 for 128 -> 256, 0.84 for 256 -> 256 and 0.77 with a skip up to t64 100;
//    1.6, 1.5, 1.23, 1.05 and 0.97 up to 256; 1.66, 1.57, 1.3, 1.2 and 1.16 above, 4 to 7
//    us each. The 256 x 64 tiles of one step (128 -> 320) 0.81, 1.06 and 1.12;
//  * 64- and 128-channel layers of 4 bits up to t64 1100, K beyond the streaming
//    kernels' two steps: gf. 3x3 64 -> 64 P 66800 15.3 -> 10.0 (t64 2088: 14.8 ->
//    15.7), 3x3 128 -> 128 P 33400 18.3 -> 13.3, 3x3 256 -> 36 P 66800 35.7 -> 22.9;
//    above, fx 128 x 128 for 65 to 128 channels and 9 steps or more, int32 at any
//    size (3x3 256 -> 80 P 133600 54.9 -> 47.4), codes up to t64 1500 (3x3 128 -> 128
//    stride 2 P 33400 18.9 -> 13.4, P 66800 19.6 -> 21.1). 36 steps or more: fx 128 x 128
//    for 65 to 128 channels at any size and of either width (3x3 512 -> 128 at t64 800:
//    0.42 of own, gf 0.66; P 416000 224 -> 169), 256-channel tiles for 129 to 255 of 4
//    bits (512 -> 192 t64 600: 0.44, 128 x 128 0.51, gf 0.65), gf for up to 64 channels to t64 2000 (512
//    -> 64 t64 1500: 0.85 of own, 2500: 1.08), at 2 bits at any size;
//  * 256-channel tiles of 4 bits, 9 steps or more: fx 256 x 128, 256 x 64 while that
//    leaves the chip short of tiles. 3x3 256 -> 256 P 133600 73.9 -> 57.9, P 16700
//    23.9 -> 16.5; 3x3 512 -> 512 P 8400 39.9 -> 25.0, P 4200 22.6 -> 17.4; 3x3 256 ->
//    720 int32 P 133600 225 -> 175; 1x1 2048 -> 512 P 8400 20.8 -> 15.2. 8 steps: fx
//    up to t64 1100 (1x1 1024 -> 256 P 16800 12.6 -> 10.4, P 33600 13.9 -> 15.1).
//    One-round launches of the 256 x 144 tiles stay (P 33600 22.5 -> 23.6);
//  * 2 bits (half the int8 kernels' time or less everywhere but in 1x1 layers of few
//    channels on many pixels and 64-channel int32 layers): gf up to 64 channels (3x3 64 ->
//    64 P 534400 37.4 -> 32.3), 1x1 layers of up to 256 channels in, 512 with a skip, only
//    to t64 1100, 2000 from 192 channels in on (gf over own for 64 -> 64 1.02 at 800, 1.11
//    at 1100, 1.6 at 3000; 256 -> 64 0.76, 0.9, 1.26), up to t64 1100 for 65 to 128, and
//    for int32 skips (1x1 256 -> 1024 P 33600 75.9 -> 56.3); else fx: 3x3 128 -> 128 P
//    133600 35.2 -> 20.7 (128 x 128), 3x3 256 -> 256 P 267200 96 -> 79.5 (256 x 128),
//    P 33600 21.8 -> 16.2 (256 x 64), 1x1 512 -> 128 P 133600 24.2 -> 14.9; 1x1 layers
//    with a skip and up to 8 steps on 128 x 128 from t64 2000 on (over own, 256 x 64 and 128 x 128: 512 -> 512
//    0.89, 0.81; 256 -> 256 t64 4000 0.96, 0.85), from 1100 on where 256-channel tiles would
//    be a quarter or more padding (512 -> 320 0.79, 0.65), and then int32 outputs from 1500 on
//    (128 -> 320 1.03, 0.94; t64 3000 1.08, 0.87).
bool plan_gf(int count, const qconv_seg_t *segs, const SegCheck *chk, int own, MfmaArgs *out, GfPlan *plan)
{
    const qconv_s &h0 = *segs[0].conv;
    if (h0.gf_kind == GF_NONE)
        return false;
    const int steps = h0.gf_steps, cout = h0.d.cout;
    const bool f4 = h0.gf_kind == GF_F4, codes = h0.d.out_mode == AQD_OUT_CODES, mfma = own >= 0;
    long long t64 = 0, pixels = 0, vpixels = 0;   // vpixels: with fx3's rows and columns of padding
    for (int i = 0; i < count; ++i) {
        const long long P = (long long)segs[i].n * chk[i].ho * chk[i].wo;
        pixels += P;
        vpixels += (long long)segs[i].n * (segs[i].h + 1) * (segs[i].w + 1);
        if (segs[i].conv->gf_kind != h0.gf_kind || chk[i].xbytes >= (1ull << 31) || P + 256 >= (1LL << 31))
            return false;   // (32-bit buffer offsets and pixel numbers)
        t64 += (P + 63) / 64 * h0.gf_groups;
    }
    const bool narrow = h0.tile_cfg == TILE_128x256 || h0.tile_cfg == TILE_64x512;
    // waves along channels and column tiles of the tiled kernels; kw 0: fx, -1: fx3
    int wc = 0, nj = 4, kw = 0;
    const bool tiled = h0.gf_kind != GF_I8 &&
                       (codes ? cout % 16 == 0 && h0.d.bits_out == h0.d.bits_in &&
                                    (h0.d.skip_bits == 0 || h0.d.skip_bits == h0.d.bits_in)
                              : cout % 4 == 0);
    const bool skip = h0.d.skip_bits != 0;
    const int cin = h0.d.cin;
    // most that fx3's pixels with padding may be, in percent of the pixels
    const bool plain = codes && !skip, one = h0.d.kh == 1 && h0.d.kw == 1;
    const bool few = one && cin <= (skip ? 512 : 256);   // (2 bits) so few K steps that own is faster on many pixels
    const int pad_limit = cin > 256 || (cin == 256 && cout <= 64)                           ? 120
                          : cin <= 128 && (cin == 64 || cout <= 128) && plain && t64 <= 2000 ? 160
                          : cout <= 128                                                     ? (plain || t64 <= 2000 ? 150 : 120)
                          : cin == 256                                                      ? 125
                                                                                            : 133;
    // 1x1 layers of up to 256 channels on persistent tiles: gf only while its tiles are few
    const bool stream = own == TILE_STREAM || own == TILE_STREAM_H128 || own == TILE_STREAM_C128 ||
                        own == TILE_STREAM_C64 || own == TILE_WVS;
    int gf_limit = 512;
    if (stream)
        gf_limit = cin == 64 || (cin == 128 && cout <= 128) ? 0 : cin == 256 && skip ? 256 : 100;
    else if (own == TILE_256x64S && steps == 1)
        gf_limit = 100;
    bool gf = false;
    if (tiled && t64 > (cin >= 256 ? 512 : 200) && h0.d.kh == 3 && h0.d.kw == 3 && h0.d.stride == 1 && h0.d.pad == 1 &&
        (cin == 64 || cin == 128 || cin % 256 == 0) && !(cin >= 256 && cout <= 64 && t64 <= 1100) &&
        !(cin > 256 && cout <= 128) && 100 * vpixels <= pad_limit * pixels) {
        kw = -1;
        if (cin == 64)
            wc = 1;
        else if (cin > 256)
            wc = 4;
        else if (cin == 128 || cout <= 128)
            wc = 2;
        else if (f4) {
            wc = !skip && t64 > (codes ? 15000 : 2500) ? 4 : 2;
            nj = wc == 4 ? 8 : 4;
        } else {
            wc = skip && t64 <= 1500 ? 2 : 4;
            nj = !skip && t64 > 1000 ? 8 : 4;
        }
    } else if (!mfma || t64 <= gf_limit) {
        gf = true;
    } else if (tiled && cout > 64 && steps >= 36 && (cout <= 128 || (!f4 && narrow))) {
        wc = cout <= 128 ? 2 : 4;
        nj = wc == 4 && t64 > 1024 && !skip ? 8 : 4;
    } else if (f4 && (h0.d.skip_bits == 32 ||
                      (cout <= 64 && (codes ? !few || t64 <= (cin <= 128 ? 1100 : 2000) : steps >= 36 || t64 <= 1100)) ||
                      (cout <= 128 && t64 <= 1100))) {
        gf = true;
    } else if (h0.gf_kind == GF_F6 && narrow && steps > 2 && t64 <= (steps >= 36 && cout <= 64 ? 2000 : 1100)) {
        gf = true;
    } else if (tiled && f4 && cout > 64 && !(cin == 64 && one && t64 > 8000)) {
        const int g = h0.gf_groups;
        const bool padded = (g + 3) / 4 * 2 > (g + 1) / 2;   // more tiles' worth of channels by fours than by twos
        wc = cout <= 128 || (one && skip && (padded ? t64 > 1100 : t64 > 2000 && steps <= 8)) || (one && !codes && padded && t64 > 1500) ? 2 : 4;
        nj = wc == 4 && t64 > (codes ? 12000 : 4000) ? 8 : 4;
    } else if (tiled && !f4 && narrow && cout > 64 && steps >= 9 && (!codes || t64 <= 1500)) {
        wc = 2;
    } else if (tiled && !f4 && !narrow && own != TILE_WV144 && (steps >= 9 || (steps == 8 && t64 <= 1100 && !skip))) {
        wc = 4;
        nj = t64 > 1024 && !skip ? 8 : 4;
    } else {
        return false;
    }
    if (!gf)
        *plan = GfPlan{h0.gf_kind, wc, nj, kw};
    else {
        // the waves of a tile split its K range while there are too few tiles to
        // give every SIMD two waves; very few tiles are halved as well. 3x3 128 ->
        // 128 P 16700 (522 tiles), 1 / 2 / 4 waves: 9.9 / 9.1 / 11.1 us; 3x3 64 -> 64
        // P 66800 (1044): 10.0 / 12.3 / 13.1; 3x3 256 -> 256 P 4200 (264): 12.7 / 12.7 /
        // 11.3; 3x3 stride 2 256 -> 256 P 77 (8): 11.9 / 8.1 / 7.2, halved 6.2, quartered
        // 5.2; 2048 -> 256 P 273 (20) 28.2, 20.7, 15.8; 3x3 256 -> 256 P 1050 (68): 7.8, 6.5,
        // 7.4
        *plan = GfPlan{h0.gf_kind, t64 <= 64 && steps >= 4 ? 2 : 4, t64 <= 100 ? 2 : 4, t64 > 1000 ? 1 : t64 > 400 ? 2 : 4};
        if (cout <= 4)   // one row tile holds every channel
            *plan = GfPlan{h0.gf_kind, 1, 4, 4};
        else if (steps < plan->kw)
            plan->kw = steps < 2 ? 1 : 2;
    }
    const int groups = wc ? (h0.gf_groups + wc - 1) / wc : cout <= 4 ? 1 : h0.gf_groups * (4 / plan->mi);
    const int px = wc ? 16 * nj * (4 / wc) : 16 * plan->nj;
    MfmaArgs &a = *out;
    a = MfmaArgs{};
    bool f32 = codes;   // fp32 requantisation when every segment has it
    for (int i = 0; i < count; ++i)
        f32 = f32 && (segs[i].n == 0 || segs[i].conv->gf_fast[segs[i].level] == 2);
    long long tiles = 0;
    for (int i = 0; i < count; ++i) {
        const qconv_seg_t &s = segs[i];
        if (s.n == 0)
            continue;
        MfmaSeg &m = a.seg[a.nseg++];
        m.x = (const uint8_t *)s.x;
        m.skip = s.skip;
        m.y = s.y;
        m.wt = (const int8_t *)s.conv->gf_w;
        m.epi = s.conv->gf_epi + (size_t)s.level * EPI_FIELDS * 64 * s.conv->gf_groups;
        m.P = (long long)s.n * chk[i].ho * chk[i].wo;
        m.n = s.n;
        m.h = s.h;
        m.w = s.w;
        m.ho = chk[i].ho;
        m.wo = chk[i].wo;
        m.hs = s.hs;
        m.ws = s.ws;
        m.tile_begin = (int)tiles;
        m.fast = f32 ? 2 : s.conv->gf_fast[s.level] ? 1 : 0;
        m.side0 = s.conv->side0[s.level];
        if (s.conv->lut_dev)
            m.lut = (f32 ? s.conv->gf_lutf : s.conv->lut_dev) + (size_t)s.level * s.conv->cout_pad * (1 << h0.d.skip_bits);
        const long long vp = plan->kw < 0 ? (long long)s.n * (s.h + 1) * (s.w + 1) : m.P;  // virtual pixels
        tiles += (vp + px - 1) / px * groups;
        if (tiles >= (1LL << 26))
            return false;
    }
    a.total_tiles = (int)tiles;
    a.tiles_per_xcd = (a.total_tiles + 7) / 8;
    a.ksplit = 1;
    a.cin = h0.d.cin;
    a.cout = h0.d.cout;
    a.cout_pad = 64 * h0.gf_groups;
    a.kh = h0.d.kh;
    a.kw = h0.d.kw;
    a.stride = h0.d.stride;
    a.pad = h0.d.pad;
    a.co_tiles = groups;
    a.ksteps = a.kchunk = h0.gf_steps;
    a.up2 = h0.d.skip_up2;
    a.bits_out = h0.d.out_mode == AQD_OUT_INT32 ? 32 : h0.d.bits_out;
    a.qmax = h0.qmax;
    a.skip_bits = h0.d.skip_bits;
    return true;
}

hipError_t launch_gf(const MfmaArgs &a, const GfPlan &p, hipStream_t stream)
{
    return p.kw <= 0 ? launch_qconv_fx(a, p, stream) : launch_qconv_gf(a, p, stream);
}

// Split of the K range: the number of parts minimising a simple model of the
// MI355X (256 CUs, two workgroups per CU), fitted to measured launches: a
// workgroup alone on its CU takes ~0.65 us per K step, two sharing a CU
// ~0.84 us (0.42 each), plus ~3 us of prologue and epilogue per pair of
// workgroups; the parts cost one write and one read of nparts x P x cout
// int32 (~5 TB/s) and the combining launch (~5 us). A split is taken only
// when the model gains 20%.
void plan_split(const MfmaArgs &a, int *nparts, int *kchunk)
{
    if (a.tile_cfg == TILE_256x64S || a.tile_cfg == TILE_256x64 || a.tile_cfg == TILE_STREAM ||
        a.tile_cfg == TILE_STREAM_C128 || a.tile_cfg == TILE_STREAM_C64 || a.tile_cfg == TILE_128x128_O3 ||
        a.tile_cfg == TILE_64x256_O3 || a.tile_cfg == TILE_STREAM_H128 || a.tile_cfg == TILE_WV || a.tile_cfg == TILE_WV144 || a.tile_cfg == TILE_WV64 || a.tile_cfg == TILE_WVS ||
        a.tile_cfg == TILE_STEM) {  // never split
        *nparts = 1;
        *kchunk = a.ksteps;
        return;
    }
    long long P = 0;
    for (int i = 0; i < a.nseg; ++i)
        P += a.seg[i].P;
    // FP4 handles (their launches never split; the size that they ask for stays):
    // half the MFMA time per 64-channel step, parts of whole 256-channel stages (4 steps)
    const bool fp4 = a.tile_cfg == TILE_FP4, b8 = a.tile_cfg == TILE_B8;
    const double step_scale = fp4 ? 0.5 : 1.0;
    const int align = fp4 ? 4 : b8 ? 2 : 1;
    auto cost = [&](int parts, int chunk) {
        const double units = (double)a.total_tiles * parts;
        const double per_cu = std::ceil(units / 256.0);
        double t = step_scale * chunk * (per_cu <= 1 ? 0.65 : 0.42 * per_cu) + 3.0 * std::ceil(per_cu / 2.0);
        if (parts > 1)
            t += (double)parts * P * a.cout * 8.0 / 5e6 + 5.0;
        return t;
    };
    *nparts = 1;
    *kchunk = a.ksteps;
    double best = cost(1, a.ksteps);
    static const int cand[] = {2, 3, 4, 6, 8, 12, 16};
    for (int c : cand) {
        const int chunk = ((a.ksteps + c - 1) / c + align - 1) / align * align;
        if (chunk < 2 || ((fp4 || b8) && chunk >= a.ksteps))
            break;
        const int parts = (a.ksteps + chunk - 1) / chunk;  // every part non-empty
        const double t = cost(parts, chunk);
        if (t < 0.8 * best) {
            best = t;
            *nparts = parts;
            *kchunk = chunk;
        }
    }
}

size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

size_t split_bytes(const MfmaArgs &a, int nparts)
{
    size_t b = 0;
    for (int i = 0; i < a.nseg; ++i)
        b += align256((size_t)nparts * a.seg[i].P * a.cout * 4);
    return b;
}

}  // namespace

extern "C" {

aqd_status_t qconv_group_workspace(int count, const qconv_seg_t *segs, size_t *bytes)
{
    REQUIRE(bytes, "null bytes");
    *bytes = 0;
    SegCheck chk[AQD_MAX_SEGS];
    MfmaArgs a;
    bool direct = false;
    aqd_status_t st = prepare_group(count, segs, chk, &a, &direct);
    if (st != AQD_OK || direct || a.nseg == 0)
        return st;
    int nparts = 1, kchunk = 0;
    plan_split(a, &nparts, &kchunk);
    if (nparts > 1)
        *bytes = split_bytes(a, nparts);
    return AQD_OK;
}

}  // extern "C"

// Scratch of qconv_run_group_static: the split-K partial sums of callers that
// cannot allocate. Every GPU the library runs on holds its own copy until the
// process ends; host code reaches it only through the per-device address from
// hipGetSymbolAddress (the array's name is a host-side stand-in).
static __device__ __align__(256) uint8_t scratch[AQD_STATIC_SCRATCH_BYTES];

namespace {

std::mutex g_scratch_mu;
void *g_scratch[64] = {};

// Device address of the current device's scratch, looked up once per device
// (with that device current); nullptr if the lookup fails.
void *static_scratch()
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64)
        return nullptr;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch[dev]) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) {
            (void)hipGetLastError();
            return nullptr;
        }
        g_scratch[dev] = p;
    }
    return g_scratch[dev];
}

// A group launch; the split-K partial sums go to `workspace` (the caller's,
// ws_bytes long, or null: no split), or with use_static to this device's
// scratch array (no allocation).
aqd_status_t run_group(int count, const qconv_seg_t *segs, void *workspace, size_t ws_bytes,
                       bool use_static, hipStream_t stream)
{
    SegCheck chk[AQD_MAX_SEGS];
    MfmaArgs a;
    bool direct = false;
    aqd_status_t st = prepare_group(count, segs, chk, &a, &direct);
    if (st != AQD_OK)
        return st;
    MfmaArgs ga;
    GfPlan gp;
    const bool gf = plan_gf(count, segs, chk, direct ? -1 : a.tile_cfg, &ga, &gp);
    if (direct && gf) {
        if (ga.nseg && launch_gf(ga, gp, stream) != hipSuccess)
            return fail(AQD_ERR_DEVICE, "global-fed conv launch failed");
        return AQD_OK;
    }
    if (direct) {
        for (int i = 0; i < count; ++i)
            if (segs[i].n > 0) {
                st = launch_direct(segs[i], chk[i], stream);
                if (st != AQD_OK)
                    return st;
            }
        return AQD_OK;
    }
    if (a.nseg == 0)
        return AQD_OK;
    const qconv_s &h0 = *segs[0].conv;
    int nparts = 1, kchunk = a.ksteps;
    if (use_static) {
        plan_split(a, &nparts, &kchunk);
        if (nparts > 1) {
            const size_t need = split_bytes(a, nparts);
            if (need > AQD_STATIC_SCRATCH_BYTES)
                return fail(AQD_ERR_UNSUPPORTED,
                            "this group's split K reduction needs " + std::to_string(need) +
                                " bytes of scratch, more than the " +
                                std::to_string((size_t)AQD_STATIC_SCRATCH_BYTES) +
                                " of the static scratch; use qconv_run_group_ws with a workspace");
            workspace = static_scratch();
            if (!workspace)
                return fail(AQD_ERR_DEVICE, "the address of the static scratch could not be found");
        }
    } else if (workspace) {
        REQUIRE(((uintptr_t)workspace & 255) == 0, "workspace must be 256-byte aligned");
        plan_split(a, &nparts, &kchunk);
        if (nparts > 1 && ws_bytes < split_bytes(a, nparts))
            nparts = 1;
    }
    if (gf) {
        if (launch_gf(ga, gp, stream) != hipSuccess)
            return fail(AQD_ERR_DEVICE, "global-fed conv launch failed");
        return AQD_OK;
    }
    if (nparts == 1) {
        if (launch_qconv_mfma(h0.d.bits_in, a, stream) != hipSuccess)
            return fail(AQD_ERR_DEVICE, "MFMA conv launch failed");
        return AQD_OK;
    }
    // part sums of every segment into its workspace slice, then the combining epilogue
    SplitArgs e{};
    e.nseg = a.nseg;
    e.nparts = nparts;
    e.cout = a.cout;
    e.cout_pad = a.cout_pad;
    e.bits_out = a.bits_out;
    e.qmax = a.qmax;
    e.skip_bits = a.skip_bits;
    e.up2 = a.up2;
    const int cpt = a.bits_out == 32 ? 4 : 32 / a.bits_out;
    uint8_t *ws = (uint8_t *)workspace;
    long long items = 0;
    for (int i = 0; i < a.nseg; ++i) {
        MfmaSeg &m = a.seg[i];
        SplitSeg &q = e.seg[i];
        q.part = (const int32_t *)ws;
        q.skip = m.skip;
        q.y = m.y;
        q.epi = m.epi;
        q.P = m.P;
        q.ho = m.ho;
        q.wo = m.wo;
        q.hs = m.hs;
        q.ws = m.ws;
        q.item_begin = items;
        items += m.P * (a.cout / cpt);
        m.y = ws;
        m.skip = nullptr;
        ws += align256((size_t)nparts * m.P * a.cout * 4);
    }
    e.total_items = items;
    a.part = 1;
    a.ksplit = nparts;
    a.kchunk = kchunk;
    a.total_tiles *= nparts;
    a.tiles_per_xcd = (a.total_tiles + 7) / 8;
    a.bits_out = 32;
    a.skip_bits = 0;
    a.up2 = 0;
    if (launch_qconv_mfma(h0.d.bits_in, a, stream) != hipSuccess)
        return fail(AQD_ERR_DEVICE, "MFMA conv launch failed");
    if (launch_splitk_epilogue(e, stream) != hipSuccess)
        return fail(AQD_ERR_DEVICE, "split-K epilogue launch failed");
    return AQD_OK;
}

}  // namespace

extern "C" {

aqd_status_t qconv_run_group_ws(int count, const qconv_seg_t *segs, void *workspace, size_t ws_bytes,
                                aqd_stream_t stream)
{
    return run_group(count, segs, workspace, ws_bytes, false, (hipStream_t)stream);
}

aqd_status_t qconv_run_group_static(int count, const qconv_seg_t *segs, aqd_stream_t stream)
{
    return run_group(count, segs, nullptr, 0, true, (hipStream_t)stream);
}

aqd_status_t qconv_run_group(int count, const qconv_seg_t *segs, aqd_stream_t stream)
{
    return run_group(count, segs, nullptr, 0, false, (hipStream_t)stream);
}

aqd_status_t qconv_run_proj(qconv_t conv, qconv_t proj, int level, int n, int h, int w,
                            const void *x, int hp, int wp, const void *xp, void *y,
                            aqd_stream_t stream_)
{
    REQUIRE(conv && proj, "null handle");
    const qconv_desc_t &d = conv->d, &e = proj->d;
    REQUIRE(level >= 0 && level < d.num_levels && level < e.num_levels, "level out of range");
    REQUIRE(n >= 0, "n must be >= 0");
    int ho = 0, wo = 0, hpo = 0, wpo = 0;
    aqd_status_t st = qconv_out_shape(conv, h, w, &ho, &wo);
    if (st != AQD_OK)
        return st;
    st = qconv_out_shape(proj, hp, wp, &hpo, &wpo);
    if (st != AQD_OK)
        return st;
    REQUIRE(hpo == ho && wpo == wo, "the projection's output size differs from the convolution's");
    REQUIRE((long long)n * ho * wo < (1LL << 31) && (long long)n * h * w < (1LL << 31) &&
                (long long)n * hp * wp < (1LL << 31),
            "too many pixels for one call");
    if (!(conv->mfma && proj->mfma && d.out_mode == AQD_OUT_CODES && d.skip_bits == 32 && !d.skip_up2 &&
          e.out_mode == AQD_OUT_INT32 && e.skip_bits == 0 && e.kh == 1 && e.kw == 1 && e.pad == 0 &&
          d.bits_in == 4 && e.bits_in == 4 && d.bits_out == 4 && d.cout == e.cout &&
          conv->tile_cfg == TILE_256x128 && proj->tile_cfg == TILE_256x128))
        return fail(AQD_ERR_UNSUPPORTED, "this pair of handles has no fused launch; run them separately");
    if (n == 0)
        return AQD_OK;
    REQUIRE(x && xp && y, "null tensor");
    REQUIRE(aligned16(x) && aligned16(xp) && aligned16(y), "tensors must be 16-byte aligned");
    const size_t xbytes = (size_t)n * h * w * d.cin * d.bits_in / 8;
    const size_t pbytes = (size_t)n * hp * wp * e.cin * e.bits_in / 8;
    const size_t ybytes = (size_t)n * ho * wo * d.cout * d.bits_out / 8;
    REQUIRE(!overlap(y, ybytes, x, xbytes) && !overlap(y, ybytes, xp, pbytes),
            "output overlaps an input");
    MfmaArgs a{};
    a.nseg = 1;
    MfmaSeg &m = a.seg[0];
    m.x = (const uint8_t *)x;
    m.skip = nullptr;
    m.y = y;
    m.wt = (const int8_t *)conv->w_dev;
    m.epi = conv->epi_dev + (size_t)level * EPI_FIELDS * conv->cout_pad;
    m.P = (long long)n * ho * wo;
    m.n = n;
    m.h = h;
    m.w = w;
    m.ho = ho;
    m.wo = wo;
    m.hs = ho;
    m.ws = wo;
    m.tile_begin = 0;
    m.fast = conv->fast[level] ? 1 : 0;   // (the projection's alignment is an integer one)
    m.side0 = 0;
    m.x2 = (const uint8_t *)xp;
    m.wt2 = (const int8_t *)proj->w_dev;
    m.epi2 = proj->epi_dev + (size_t)level * EPI_FIELDS * proj->cout_pad;
    m.h2 = hp;
    m.w2 = wp;
    const long long tiles = (m.P + PROJ_BLK_PX - 1) / PROJ_BLK_PX * conv->co_tiles;
    REQUIRE(tiles < (1LL << 26), "too many tiles for one launch");
    a.total_tiles = (int)tiles;
    a.tiles_per_xcd = (a.total_tiles + 7) / 8;
    a.ksplit = 1;
    a.kchunk = conv->ksteps;
    a.part = 0;
    a.cin = d.cin;
    a.cout = d.cout;
    a.cout_pad = conv->cout_pad;
    a.kh = d.kh;
    a.kw = d.kw;
    a.stride = d.stride;
    a.pad = d.pad;
    a.co_tiles = conv->co_tiles;
    a.ksteps = conv->ksteps;
    a.up2 = 0;
    a.tile_cfg = conv->tile_cfg;
    a.bits_out = d.bits_out;
    a.qmax = conv->qmax;
    a.skip_bits = 32;
    a.zero = conv->zero;
    a.cin2 = e.cin;
    a.stride2 = e.stride;
    a.ksteps2 = proj->ksteps;
    // one K step each (cin 64): persistent streaming tiles (same 256 x 64 tiles)
    const bool stream_tiles = conv->ksteps == 1 && proj->ksteps == 1 && d.kh == 1 && d.kw == 1 &&
                              d.pad == 0 && d.cout % 256 == 0;
    // both inputs in 256-channel chunks (the main one may have 128 channels:
    // one padded stage), 1x1 stride 1: register-fed 256 x 64 tiles (32-bit
    // buffer offsets: inputs below 2^31 bytes)
    const bool wv_tiles = (d.cin % 256 == 0 || d.cin == 128) && e.cin % 256 == 0 && d.kh == 1 && d.kw == 1 && d.stride == 1 &&
                          d.pad == 0 && xbytes < (1ull << 31) && pbytes < (1ull << 31);
    hipError_t err;
    if (stream_tiles) {
        a.tile_cfg = TILE_STREAM;
        err = launch_qconv_mfma(4, a, (hipStream_t)stream_);
    } else if (wv_tiles) {
        a.tile_cfg = TILE_WV64;
        err = launch_qconv_wv_proj(a, (hipStream_t)stream_);
    } else {
        err = launch_qconv_proj(a, (hipStream_t)stream_);
    }
    if (err != hipSuccess)
        return fail(AQD_ERR_DEVICE, "fused projection launch failed");
    return AQD_OK;
}

aqd_status_t qconv_run(qconv_t conv, int level, int n, int h, int w, const void *x, const void *skip,
                       int hs, int ws, void *y, aqd_stream_t stream)
{
    qconv_seg_t s{conv, level, n, h, w, x, skip, hs, ws, y};
    return qconv_run_group(1, &s, stream);
}

aqd_status_t qadd_run(const qadd_desc_t *desc, const void *a, const void *b, void *y,
                      const qadd_params_t *p, aqd_stream_t stream)
{
    REQUIRE(desc && p, "null argument");
    qadd_desc_t d = *desc;
    REQUIRE(d.n >= 0 && d.h >= 1 && d.w >= 1 && d.c >= 1, "bad tensor shape");
    REQUIRE(code_bits(d.bits_a) || d.bits_a == 32, "bits_a must be 2, 3, 4, 8 or 32");
    REQUIRE(code_bits(d.bits_b) || d.bits_b == 32, "bits_b must be 2, 3, 4, 8 or 32");
    REQUIRE(code_bits(d.bits_out), "bits_out must be 2, 3, 4 or 8");
    const int qmax = (1 << d.bits_out) - 1;
    d.bits_a = stored_bits(d.bits_a);  // widths as stored from here on
    d.bits_b = stored_bits(d.bits_b);
    d.bits_out = stored_bits(d.bits_out);
    REQUIRE((d.c * d.bits_a) % 8 == 0 && (d.c * d.bits_b) % 8 == 0 && (d.c * d.bits_out) % 8 == 0,
            "c * bits must be a multiple of 8");
    if (d.up2)
        REQUIRE(d.up2 == 1 && (d.h - 1) / 2 < d.hb && (d.w - 1) / 2 < d.wb && d.hb >= 1 && d.wb >= 1,
                "upsampled operand too small");
    else
        REQUIRE(d.hb == d.h && d.wb == d.w, "operand sizes differ");
    REQUIRE((long long)d.n * d.h * d.w < (1LL << 31), "too many pixels for one call");
    if (d.n == 0)
        return AQD_OK;
    REQUIRE(a && b && y, "null tensor");
    REQUIRE(aligned16(a) && aligned16(b) && aligned16(y), "tensors must be 16-byte aligned");
    REQUIRE(p->skip_c && p->skip_d && p->skip_side && p->mult && p->shift, "null parameter array");
    const size_t ab = (size_t)d.n * d.h * d.w * d.c * d.bits_a / 8;
    const size_t bb = (size_t)d.n * d.hb * d.wb * d.c * d.bits_b / 8;
    const size_t yb = (size_t)d.n * d.h * d.w * d.c * d.bits_out / 8;
    REQUIRE(!overlap(y, yb, a, ab) && !overlap(y, yb, b, bb), "output overlaps an input");
    QaddArgs q{};
    q.a = a;
    q.b = b;
    q.y = (uint8_t *)y;
    q.skip_c = p->skip_c;
    q.skip_d = p->skip_d;
    q.skip_side = p->skip_side;
    q.mult = p->mult;
    q.shift = p->shift;
    q.n = d.n;
    q.h = d.h;
    q.w = d.w;
    q.c = d.c;
    q.hb = d.hb;
    q.wb = d.wb;
    q.bits_a = d.bits_a;
    q.bits_b = d.bits_b;
    q.bits_out = d.bits_out;
    q.qmax = qmax;
    q.up2 = d.up2;
    if (launch_qadd(q, (hipStream_t)stream) != hipSuccess)
        return fail(AQD_ERR_DEVICE, "qadd launch failed");
    return AQD_OK;
}

aqd_status_t aqd_channel_sums(const int32_t *v, int64_t rows, int c, int64_t *sums,
                              aqd_stream_t stream)
{
    REQUIRE(rows >= 0 && c >= 1, "bad shape");
    if (rows == 0)
        return AQD_OK;
    REQUIRE(v && sums, "null pointer");
    if (launch_channel_sums(v, rows, c, (long long *)sums, (hipStream_t)stream) != hipSuccess)
        return fail(AQD_ERR_DEVICE, "channel sums launch failed");
    return AQD_OK;
}

aqd_status_t aqd_mfma_probe(int workgroups, int iters, int32_t *out, aqd_stream_t stream)
{
    REQUIRE(workgroups >= 1 && workgroups <= (1 << 20) && iters >= 1, "workgroups in 1..2^20, iters >= 1");
    REQUIRE(out, "null pointer");
    if (launch_mfma_probe(workgroups, iters, out, (hipStream_t)stream) != hipSuccess)
        return fail(AQD_ERR_DEVICE, "probe launch failed");
    return AQD_OK;
}

aqd_status_t aqd_maxpool_run(const aqd_maxpool_desc_t *desc, const void *x, void *y,
                             aqd_stream_t stream)
{
    REQUIRE(desc, "null argument");
    aqd_maxpool_desc_t d = *desc;
    REQUIRE(d.n >= 0 && d.h >= 1 && d.w >= 1 && d.c >= 1, "bad tensor shape");
    REQUIRE(code_bits(d.bits), "bits must be 2, 3, 4 or 8");
    d.bits = stored_bits(d.bits);
    REQUIRE((d.c * d.bits) % 8 == 0, "c * bits must be a multiple of 8");
    REQUIRE(d.k >= 1 && d.k <= 7 && d.stride >= 1 && d.stride <= 4 && d.pad >= 0 && d.pad < d.k,
            "k must be in 1..7, stride in 1..4, pad in 0..k-1");
    const int ho = (d.h + 2 * d.pad - d.k) / d.stride + 1;
    const int wo = (d.w + 2 * d.pad - d.k) / d.stride + 1;
    REQUIRE(d.h + 2 * d.pad >= d.k && d.w + 2 * d.pad >= d.k && ho >= 1 && wo >= 1,
            "input smaller than the window");
    REQUIRE((long long)d.n * d.h * d.w < (1LL << 31), "too many pixels for one call");
    if (d.n == 0)
        return AQD_OK;
    REQUIRE(x && y, "null tensor");
    const size_t xb = (size_t)d.n * d.h * d.w * d.c * d.bits / 8;
    const size_t yb = (size_t)d.n * ho * wo * d.c * d.bits / 8;
    REQUIRE(!overlap(y, yb, x, xb), "output overlaps the input");
    PoolArgs a{};
    a.x = (const uint8_t *)x;
    a.y = (uint8_t *)y;
    a.n = d.n;
    a.h = d.h;
    a.w = d.w;
    a.c = d.c;
    a.bits = d.bits;
    a.k = d.k;
    a.stride = d.stride;
    a.pad = d.pad;
    a.ho = ho;
    a.wo = wo;
    if (launch_maxpool(a, (hipStream_t)stream) != hipSuccess)
        return fail(AQD_ERR_DEVICE, "max-pooling launch failed");
    return AQD_OK;
}

// ------------------------------------------------------------------ graph capture
aqd_status_t aqd_graph_begin(aqd_stream_t stream)
{
    REQUIRE(stream, "capture needs a stream other than the null stream");
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing((hipStream_t)stream, &st) != hipSuccess)
        return fail(AQD_ERR_DEVICE, "stream query failed");
    REQUIRE(st == hipStreamCaptureStatusNone, "the stream is already capturing");
    if (hipStreamBeginCapture((hipStream_t)stream, hipStreamCaptureModeThreadLocal) != hipSuccess)
        return fail(AQD_ERR_DEVICE, "stream capture could not start");
    return AQD_OK;
}

aqd_status_t aqd_graph_end(aqd_stream_t stream, void **graph_exec)
{
    REQUIRE(stream && graph_exec, "null stream or output pointer");
    *graph_exec = nullptr;
    hipGraph_t g = nullptr;
    if (hipStreamEndCapture((hipStream_t)stream, &g) != hipSuccess || !g) {
        (void)hipGetLastError();
        return fail(AQD_ERR_DEVICE, "stream capture failed (an operation was not capturable)");
    }
    hipGraphExec_t e = nullptr;
    const hipError_t r = hipGraphInstantiate(&e, g, nullptr, nullptr, 0);
    (void)hipGraphDestroy(g);
    if (r != hipSuccess || !e)
        return fail(AQD_ERR_DEVICE, "graph instantiation failed");
    *graph_exec = (void *)e;
    return AQD_OK;
}

aqd_status_t aqd_graph_launch(void *graph_exec, aqd_stream_t stream)
{
    REQUIRE(graph_exec, "null graph");
    if (hipGraphLaunch((hipGraphExec_t)graph_exec, (hipStream_t)stream) != hipSuccess)
        return fail(AQD_ERR_DEVICE, "graph launch failed");
    return AQD_OK;
}

void aqd_graph_destroy(void *graph_exec)
{
    if (graph_exec)
        (void)hipGraphExecDestroy((hipGraphExec_t)graph_exec);
}

// ------------------------------------------------------------------ host helpers
aqd_status_t aqd_pack_codes(const uint8_t *codes, int64_t rows, int c, int bits, uint8_t *out)
{
    REQUIRE(codes && out && rows >= 0 && c >= 1 && code_bits(bits) && (c * stored_bits(bits)) % 8 == 0,
            "bad arguments");
    const int sb = stored_bits(bits);
    const int rb = c * sb / 8;
    const int mask = (1 << bits) - 1;
    for (int64_t r = 0; r < rows; ++r) {
        uint8_t *o = out + r * rb;
        std::memset(o, 0, rb);
        for (int ch = 0; ch < c; ++ch) {
            const int v = codes[r * c + ch];
            REQUIRE(v <= mask, "code out of range for the bitwidth");
            const int bit = ch * sb;
            o[bit >> 3] |= (uint8_t)(v << (bit & 7));
        }
    }
    return AQD_OK;
}

aqd_status_t aqd_unpack_codes(const uint8_t *packed, int64_t rows, int c, int bits, uint8_t *out)
{
    REQUIRE(packed && out && rows >= 0 && c >= 1 && code_bits(bits) && (c * stored_bits(bits)) % 8 == 0,
            "bad arguments");
    const int sb = stored_bits(bits);
    const int rb = c * sb / 8;
    for (int64_t r = 0; r < rows; ++r)
        for (int ch = 0; ch < c; ++ch) {
            const int bit = ch * sb;
            out[r * c + ch] = (packed[r * rb + (bit >> 3)] >> (bit & 7)) & ((1 << bits) - 1);
        }
    return AQD_OK;
}

aqd_status_t aqd_approx_ratio(double r, int32_t *c_out, int32_t *d_out)
{
    REQUIRE(c_out && d_out, "null argument");
    REQUIRE(std::isfinite(r) && r >= 1.0 && r < 1073741824.0, "ratio must be in [1, 2^30)");
    bool have = false;
    double best_err = 0.0;
    int32_t bc = 0, bd = 0;
    for (int d = 1; d <= 31; ++d) {
        const double x = std::ldexp(r, d);
        if (x + 0.5 >= 2147483648.0)
            break;
        const double c = std::floor(x + 0.5);
        const double err = std::fabs(r - std::ldexp(c, -d));
        if (!have || err < best_err) {
            have = true;
            best_err = err;
            bc = (int32_t)c;
            bd = d;
        }
    }
    *c_out = bc;
    *d_out = bd;
    return AQD_OK;
}

aqd_status_t aqd_normalize_multiplier(double r, int32_t *mult, int32_t *shift)
{
    REQUIRE(mult && shift, "null argument");
    REQUIRE(std::isfinite(r) && r != 0.0, "scale must be finite and non-zero");
    const double a = std::fabs(r);
    int e = 0;
    (void)std::frexp(a, &e);  // a = m * 2^e, m in [0.5, 1)
    int d = 31 - e;           // a * 2^d in [2^30, 2^31)
    double c = std::floor(std::ldexp(a, d) + 0.5);
    if (c == 2147483648.0) {
        c = 1073741824.0;
        d -= 1;
    }
    const int sh = d - 31;
    REQUIRE(sh >= -31 && sh <= 31, "scale out of range for the dyadic form");
    *mult = r < 0 ? -(int32_t)c : (int32_t)c;
    *shift = sh;
    return AQD_OK;
}

aqd_status_t aqd_bn_stats_from_sums(int cout, const int64_t *s1, const int64_t *s2, int64_t count,
                                    double alpha_conv, double *mean, double *var)
{
    REQUIRE(cout >= 1 && s1 && s2 && mean && var && count >= 1, "bad arguments");
    for (int i = 0; i < cout; ++i) {
        const double m = (double)s1[i] / (double)count;
        const double va = (double)s2[i] / (double)count - m * m;
        mean[i] = alpha_conv * m;
        var[i] = (alpha_conv * alpha_conv) * va;
    }
    return AQD_OK;
}

aqd_status_t aqd_fold_bn(int cout, const double *gamma, const double *beta, const double *mean,
                         const double *var, double eps, double alpha_conv, int32_t *bias,
                         double *alpha_z)
{
    REQUIRE(cout >= 1 && gamma && beta && mean && var && bias && alpha_z, "bad arguments");
    REQUIRE(std::isfinite(alpha_conv) && alpha_conv > 0.0, "alpha_conv must be positive");
    for (int i = 0; i < cout; ++i) {
        REQUIRE(gamma[i] != 0.0 && var[i] + eps > 0.0, "gamma must be non-zero and var + eps > 0");
        const double sd = std::sqrt(var[i] + eps);
        const double s = (beta[i] * sd / gamma[i] - mean[i]) / alpha_conv;
        const double rb = std::floor(s + 0.5);
        REQUIRE(rb > -2147483648.0 && rb < 2147483648.0, "folded bias outside int32");
        bias[i] = (int32_t)rb;
        alpha_z[i] = alpha_conv * gamma[i] / sd;
    }
    return AQD_OK;
}

aqd_status_t aqd_skip_params(int cout, const double *alpha_z, const double *alpha_k,
                             int alpha_k_per_channel, int32_t *c, int32_t *d, int32_t *side,
                             double *scale)
{
    REQUIRE(cout >= 1 && alpha_z && alpha_k && c && d && side && scale, "bad arguments");
    for (int i = 0; i < cout; ++i) {
        const double az = alpha_z[i];
        const double ak = alpha_k_per_channel ? alpha_k[i] : alpha_k[0];
        REQUIRE(std::isfinite(az) && std::isfinite(ak) && az != 0.0 && ak != 0.0,
                "scales must be finite and non-zero");
        // opposite signs (a normalisation with gamma < 0): the numerator is negated
        const bool neg = (az < 0.0) != (ak < 0.0);
        aqd_status_t st;
        if (std::fabs(ak) >= std::fabs(az)) {
            st = aqd_approx_ratio(std::fabs(ak / az), &c[i], &d[i]);
            side[i] = 0;
            scale[i] = az;
        } else {
            st = aqd_approx_ratio(std::fabs(az / ak), &c[i], &d[i]);
            side[i] = 1;
            scale[i] = ak;
        }
        if (st != AQD_OK)
            return st;
        if (neg)
            c[i] = -c[i];
    }
    return AQD_OK;
}

aqd_status_t aqd_requant_params(int cout, const double *scale, double alpha_out, int32_t *mult,
                                int32_t *shift)
{
    REQUIRE(cout >= 1 && scale && mult && shift, "bad arguments");
    REQUIRE(std::isfinite(alpha_out) && alpha_out > 0.0, "alpha_out must be positive");
    for (int i = 0; i < cout; ++i) {
        aqd_status_t st = aqd_normalize_multiplier(scale[i] / alpha_out, &mult[i], &shift[i]);
        if (st != AQD_OK)
            return st;
    }
    return AQD_OK;
}

}  // extern "C"
