// Implicit-GEMM integer convolution on the gfx950 block-float MFMA
// (v_mfma_f32_16x16x128_f8f6f4) with exact small-integer operands, for launches
// that fill the GPU. Kinds, operand formats, the exactness argument and the
// weight layout are those of the global-fed kernel (qconv_gf.hip): F6 = codes of
// at most 4 bits in 4-bit containers with weights of at most 4 bits as e2m3, F4 =
// 2-bit codes and weights as e2m1. The GEMM view is that of Eq. 4 (Sec. 3.2.1):
// rows = output channels, columns = output pixels, K = taps x input channels; a
// K step is 128 channels (four chunks of 32), a stage two steps.
//
// Workgroup: 4 waves, WC along channels x WP along pixels; a wave owns 64
// channels (4 row tiles) x 16 NJ pixels:
//  * weights go from global memory (L2) straight into registers, one K step
//    ahead of their MFMAs (24 bytes per lane and row tile for e2m3);
//  * activation codes go through LDS in stages of 256 channels of the K range
//    (eight chunks; a stage may span taps), widened to the MFMA's format by the
//    copy, once per workgroup instead of once per wave: 16 codes of 4 bits move
//    to 6-bit fields in 8 instructions. A pixel's chunk is 24 bytes (e2m3): 16 in
//    a 128-byte row of eight 16-byte columns, 8 in a 64-byte row of eight 8-byte
//    columns, both XOR-swizzled with the pixel so that the copies' writes and the
//    fragment reads are free of bank conflicts. Two buffers, one barrier per
//    stage: stage t + 1 is written during stage t from registers loaded during
//    stage t - 1.
// Buffer loads return zeros past a buffer's size: padding taps, pixels past the
// end and steps past the last cost no branch.
//
// What bounds it (measured on 3x3 256 -> 256 stride 1, 267200 pixels, 256 x 128 tiles, a
// layer that the 3x3 kernel below takes since: 140 us on the int8 register-fed kernel,
// 107 us here, 2940 int TOPS of the 7000 the MFMA alone reaches on these operands):
// timing variants that leave work out gain 9% without the weight loads, 19% without the
// copies' widening and LDS writes, 19% without the epilogue; matrix cores busy 32%,
// LDS 21%. What it runs now: other strides, 1x1 layers, padded images (plan_gf).
//
// Epilogue (Sec. 3.2.2-3.2.3, Eq. 6-8, Eq. 2 on integers): a lane holds 16
// consecutive channels of NJ pixels.

#include "epilogue.h"
#include "internal.h"
#include "mfma_common.h"

namespace aqd {
namespace {

typedef float v4f __attribute__((ext_vector_type(4)));

// LDS bytes the epilogue needs
template <int KIND, int WC, int NJ, int OUTK, int SKK>
constexpr int fx_epilogue_bytes()
{
    constexpr int BPX = 16 * NJ * (4 / WC), BO = KIND == GF_F6 ? 4 : 2;
    constexpr int tabs = WC * (EPI_FIELDS + (SKK == 1 ? 1 << BO : 0)) * 64 * 4;
    constexpr int outb = OUTK == 1 ? 64 * WC * 64 * 4 : BPX * WC * 64 * BO / 8;
    return OUTK == 1 || outb > tabs ? outb : tabs;
}

// With fp32 requantisation and no skip the epilogue reads two numbers per channel:
// their copy to LDS (2 x 64 WC words at ftab) starts with the kernel and has long
// landed by the end of the K loop, where loading the tables would keep the tile's
// waves waiting twice (3x3 256 -> 256 on 267200 pixels: 88.8 -> 86.5 us, 128 ->
// 128 on 133600: 21.2 -> 20.0). Every lane
// waits for later loads of its own before the barrier that follows.
template <int WC>
__device__ __forceinline__ void fx_early_table(const MfmaArgs &A, const MfmaSeg &S, const int32_t *ftab, int co_tile,
                                               int tid)
{
    static_assert(EPI_FB == EPI_FA + 1, "fields in order");
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (wave < 2 && lane < 16 * WC) {
        // (a partial last channel tile: the table's own last channels again)
        const int c = min(co_tile * (WC * 64) + 4 * lane, A.cout_pad - 4);
        dma16(S.epi + (EPI_FA + wave) * A.cout_pad + c, lds_addr(ftab) + wave * (WC * 256));
    }
}

// The epilogue of both tiled kernels: accumulators -> outputs. pixel(p): output
// pixel of the tile's pixel p (wave wp's column j: pixels 16 (NJ wp + j) + r), or
// -1. lds: fx_epilogue_bytes, free once every wave has arrived here. ftab: a and b of
// the tile's channels (fx_early_table), where the epilogue needs no other table.
template <int KIND, int WC, int NJ, int OUTK, int SKK, int FAST, typename PX>
__device__ __forceinline__ void fx_epilogue(const MfmaArgs &A, const MfmaSeg &S, uint8_t *lds, const int32_t *ftab,
                                            v4f (&acc)[4][NJ], const int co_tile, const int tid, PX &&pixel)
{
    constexpr bool F6 = KIND == GF_F6;
    constexpr int MI = 4, BPX = 16 * NJ * (4 / WC);
    constexpr int BO = F6 ? 4 : 2, QMAX = (1 << BO) - 1;   // output code width
    constexpr bool EARLY = FAST == 2 && SKK == 0;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wc = wave % WC, wp = wave / WC, r = lane & 15, g = lane >> 4;
    const int pw = 16 * NJ * wp + r;
    const int ct = co_tile * WC + wc, groups = A.cout_pad / 64, hw = S.ho * S.wo;
    constexpr float UNIT = F6 ? 64.f : 2.f;
    const int c0 = 64 * ct + 16 * g;                 // first of this lane's 16 channels
    if constexpr (OUTK == 1) {
        // int32 outputs, 64 pixels of the tile at a time: each lane's 16 channels
        // go to LDS rows of WC * 64 int32 (16-byte chunk c of pixel p at
        // c ^ (p & 7)), then every thread stores 16-byte chunks of whole rows
        constexpr int CH = WC * 16;                  // chunks per row
        v4i bias[MI];
#pragma unroll
        for (int i = 0; i < MI; ++i)
            bias[i] = ct < groups ? *(const v4i *)(S.epi + EPI_BIAS * A.cout_pad + c0 + 4 * i) : v4i{0, 0, 0, 0};
        const int valid = min(A.cout - co_tile * (WC * 64), WC * 64) / 4;
        static_for<BPX / 64>([&](auto pc) {
            constexpr int pass = decltype(pc)::value;
            __syncthreads();   // the ring, or the last pass's rows, are no longer read
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                // this wave's column j is pixels 16 (NJ wp + j) .. of the tile
                if ((NJ * wp + j) / 4 == pass) {
                    const int p = (16 * (NJ * wp + j)) % 64 + r;
#pragma unroll
                    for (int i = 0; i < MI; ++i) {
                        const int c = 16 * wc + 4 * g + i;
                        const v4f a = acc[i][j];
                        *(v4i *)(lds + (p * CH + (c ^ (p & 7))) * 16) =
                            v4i{(int)(a.x * UNIT), (int)(a.y * UNIT), (int)(a.z * UNIT), (int)(a.w * UNIT)} + bias[i];
                    }
                }
            }
            __syncthreads();
#pragma unroll
            for (int it = 0; it < CH / 4; ++it) {
                const int idx = it * 256 + tid;
                const int p = idx / CH, c = idx % CH;
                const long long px = pixel(64 * pass + p);
                if (px >= 0 && c < valid)
                    *(v4i *)((int32_t *)S.y + px * A.cout + co_tile * (WC * 64) + 4 * c) =
                        *(const v4i *)(lds + (p * CH + (c ^ (p & 7))) * 16);
            }
        });
        return;
    }

    // ---------------------------------------------------------------- epilogue
    constexpr int OW = BO / 2;                       // words of a lane's 16 channels
    const bool co_ok = c0 < A.cout;                  // (cout is a multiple of 16: all 16 or none)
    uint32_t skw[NJ][OW];
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
#pragma unroll
        for (int o = 0; o < OW; ++o)
            skw[j][o] = 0;
        if constexpr (SKK == 1) {
            const long long px = pixel(pw + 16 * j);
            if (co_ok && px >= 0) {
                long long spix = px;
                if (A.up2) {
                    const unsigned pn = (unsigned)px / (unsigned)hw, prem = (unsigned)px - pn * (unsigned)hw;
                    const unsigned oh = prem / (unsigned)S.wo, ow = prem - oh * (unsigned)S.wo;
                    spix = ((long long)pn * S.hs + (oh >> 1)) * S.ws + (ow >> 1);
                }
                const uint8_t *src = (const uint8_t *)S.skip + (spix * A.cout + c0) * BO / 8;
                load_words<OW>(src, skw[j]);
            }
        }
    }
    // the tables of the tile's channels, and of side-0 skips RSM(k, c, d) per code
    int32_t *prm = (int32_t *)lds;                   // [EPI_FIELDS][WC * 64]
    int32_t *lut = prm + EPI_FIELDS * WC * 64;       // [WC * 64][QMAX + 1]
    const bool use_lut = SKK == 1 && S.side0;
    if constexpr (!EARLY) {
        __syncthreads();   // every wave is done with the ring
        for (int u = tid; u < EPI_FIELDS * WC * 64; u += 256) {
            const int f = u / (WC * 64), c = u % (WC * 64);
            prm[u] = co_tile * (WC * 64) + c < A.cout_pad ? S.epi[f * A.cout_pad + co_tile * (WC * 64) + c] : 0;
        }
        if (use_lut)
            for (int u = tid; u < WC * 64 * (QMAX + 1); u += 256)
                lut[u] = co_tile * (WC * 64) + u / (QMAX + 1) < A.cout
                             ? S.lut[(long long)co_tile * (WC * 64) * (QMAX + 1) + u] : 0;
        __syncthreads();
    }
    uint32_t outw[NJ][OW];
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int o = 0; o < OW; ++o)
            outw[j][o] = 0;
    const int cl = 64 * wc + 16 * g;
    const int32_t *lut_l = lut + cl * (QMAX + 1);
    auto group = [&](auto lut_c, auto ic) {
        constexpr bool LUT = decltype(lut_c)::value;
        constexpr int i = decltype(ic)::value;
        const int32_t *tab = (EARLY ? ftab - EPI_FA * WC * 64 : prm) + cl + 4 * i;
        v4i bias = {0, 0, 0, 0};
        if constexpr (FAST != 2)
            bias = *(const v4i *)(tab + EPI_BIAS * WC * 64);
        const v4i mult = *(const v4i *)(tab + (FAST == 2 ? EPI_FB : EPI_MULT) * WC * 64);
        const v4i shf = *(const v4i *)(tab + (FAST == 2 ? EPI_FA : EPI_SHIFT) * WC * 64);
        v4i sc = {0, 0, 0, 0}, sd = sc, ss = sc;
        long long srnd[4] = {0, 0, 0, 0};
        if constexpr (SKK != 0 && !LUT) {
            sc = *(const v4i *)(tab + EPI_SKIP_C * WC * 64);
            sd = *(const v4i *)(tab + EPI_SKIP_D * WC * 64);
            ss = *(const v4i *)(tab + EPI_SKIP_SIDE * WC * 64);
#pragma unroll
            for (int e = 0; e < 4; ++e)
                srnd[e] = rsm_rnd(sd[e]);
        }
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int v = FAST == 2 ? 0 : (int)(acc[i][j][e] * UNIT) + bias[e];
                const int bit = (4 * i + e) * BO;
                int kv = 0;
                if constexpr (SKK == 1)
                    kv = (int)__builtin_amdgcn_ubfe(skw[j][bit >> 5], bit & 31, BO);
                int y;
                if constexpr (FAST == 2) {   // the accumulator itself: the tables hold the bias and its unit
                    float b = __int_as_float(mult[e]);
                    if constexpr (LUT)
                        b = __int_as_float(lut_l[(4 * i + e) * (QMAX + 1) + kv]);
                    y = quant_f32(acc[i][j][e], __int_as_float(shf[e]), b, (float)QMAX);
                } else if constexpr (FAST) {
                    int u = v;
                    if constexpr (LUT) {
                        u = (int)((unsigned)v + (unsigned)lut_l[(4 * i + e) * (QMAX + 1) + kv]);
                    } else if constexpr (SKK != 0) {
                        const int scaled = rsm32r(ss[e] ? v : kv, sc[e], srnd[e], sd[e]);
                        u = (int)((unsigned)scaled + (unsigned)(ss[e] ? kv : v));
                    }
                    y = requant32(u, mult[e], requant_rnd(shf[e]), shf[e] - 1);
                    y = y < 0 ? 0 : (y > QMAX ? QMAX : y);
                } else {
                    long long u = v;
                    if constexpr (LUT)
                        u = (int)((unsigned)v + (unsigned)lut_l[(4 * i + e) * (QMAX + 1) + kv]);
                    else if constexpr (SKK != 0)
                        u = align_add(v, kv, sc[e], sd[e], ss[e]);
                    y = (int)requant_clamp(u, mult[e], shf[e], QMAX);
                    asm volatile("" : "+v"(y));   // one 64-bit product alive at a time
                }
                outw[j][bit >> 5] |= (uint32_t)y << (bit & 31);
            }
        }
    };
    if (FAST == 2 ? SKK == 1 : use_lut)
        static_for<MI>([&](auto ic) { group(std::integral_constant<bool, SKK == 1>{}, ic); });
    else if constexpr (FAST != 2 || SKK != 1)
        static_for<MI>([&](auto ic) { group(std::false_type{}, ic); });
    if (F6 && A.qmax == 7) {   // 3-bit codes (clamped to 15 above)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int o = 0; o < OW; ++o)
                outw[j][o] = sat7_nibbles(outw[j][o]);
    }
    // the packed words are complete here (see the fences of the other kernels)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int o = 0; o < OW; ++o)
            asm volatile("" : "+v"(outw[j][o]));
    // a whole channel tile's codes go through LDS and out as 16-byte chunks of
    // contiguous pixel rows; a partial one is stored from registers
    constexpr int ROWB = WC * 64 * BO / 8, CPR = ROWB / 16;
    if (A.cout - co_tile * (WC * 64) >= WC * 64) {
        __syncthreads();
        const int cb = cl * BO / 8;
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const int p = pw + 16 * j;
            uint8_t *d = lds + p * ROWB + 16 * ((cb >> 4) ^ (p & (CPR - 1))) + (cb & 15);
            store_words<OW>(d, outw[j]);
        }
        __syncthreads();
        const long long rowg = (long long)A.cout * BO / 8;
#pragma unroll
        for (int it = 0; it < (BPX * CPR + 255) / 256; ++it) {
            const int idx = it * 256 + tid;
            const int p = idx / CPR, c = idx % CPR;
            const long long px = p < BPX ? pixel(p) : -1;
            if (px >= 0)
                *(uint4 *)((uint8_t *)S.y + px * rowg + co_tile * ROWB + 16 * c) =
                    *(const uint4 *)(lds + p * ROWB + 16 * (c ^ (p & (CPR - 1))));
        }
        return;
    }
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const long long px = pixel(pw + 16 * j);
        if (co_ok && px >= 0)
            store_words<OW>((uint8_t *)S.y + (px * A.cout + c0) * BO / 8, outw[j]);
    }
}


// OUTK: 0 = codes of the input's width, 1 = int32; SKK: 0 = none, 1 = codes of
// the input's width; FAST: 1 = every shift >= 2 (32-bit requantisation), 2 = fp32
// requantisation (skips: all of side 0); OCC:
// workgroups per CU
template <int KIND, int WC, int NJ, int OUTK, int SKK, int FAST, int OCC>
__global__ void __launch_bounds__(256, OCC) qconv_fx_kernel(MfmaArgs A)
{
    constexpr bool F6 = KIND == GF_F6;
    constexpr int WP = 4 / WC, MI = 4;
    constexpr int BPX = 16 * NJ * WP;                // pixels per workgroup tile
    constexpr int NPC = BPX / 32;                    // copy pieces of 32 pixels per stage
    constexpr int PPS = (NPC + 1) / 2;               // pieces per K step
    constexpr int XB = F6 ? 16 : 8;                  // packed bytes of a chunk
    constexpr int WB = F6 ? GF_F6_TILE : 1024;       // weight bytes of a row tile and K step
    constexpr int XROW = 128, YROW = F6 ? 64 : 0;    // LDS bytes of a pixel and stage
    constexpr int STAGE = BPX * (XROW + YROW);
    constexpr int EPIB = fx_epilogue_bytes<KIND, WC, NJ, OUTK, SKK>();
    constexpr bool EARLY = FAST == 2 && SKK == 0 && OUTK == 0;
    constexpr int OFF_F = 2 * STAGE > EPIB ? 2 * STAGE : EPIB;
    constexpr int LDS = OFF_F + (EARLY ? 2 * WC * 256 : 0);
    constexpr int RA = NJ >= 8 ? 2 : 1;              // fragments are read RA column tiles ahead
    static_assert(NJ >= 4 && NPC >= 2 && NPC <= 8, "tile");
    __shared__ __attribute__((aligned(1024))) uint8_t lds[LDS];

    const int bid = blockIdx.x;
    const int tile = (bid & 7) * A.tiles_per_xcd + (bid >> 3);
    if (tile >= A.total_tiles)
        return;
    int s = 0;
    if (A.nseg > 1) {
#pragma unroll
        for (int i = 1; i < AQD_MAX_SEGS; ++i)
            if (i < A.nseg && tile >= A.seg[i].tile_begin)
                s = i;
    }
    const MfmaSeg &S = A.seg[s];
    const int t_in_seg = tile - S.tile_begin;
    const int co_tile = t_in_seg % A.co_tiles;
    const int px_tile = t_in_seg / A.co_tiles;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wc = wave % WC, wp = wave / WC;
    const int r = lane & 15, g = lane >> 4;
    const int KS = A.ksteps;                         // K steps (of 128 channels)
    const int NST = (KS + 1) / 2;
    const int hw = S.ho * S.wo;
    const int32_t *const ftab = (const int32_t *)(lds + OFF_F % LDS);
    if constexpr (EARLY)
        fx_early_table<WC>(A, S, ftab, co_tile, tid);

    // ---- activation copies: piece m of a stage = pixels 32m .. 32m+31 of the
    // tile, lane tid copying chunk tid % 8 of the stage for pixel 32m + tid / 8;
    // per piece the byte offset of the pixel's window origin and which window
    // rows (bit t) and columns (bit 16 + t) lie inside the image
    const int c8 = tid & 7, cp = tid >> 3;
    const int row_bytes = A.cin * XB / 32;
    int xbase[NPC];
    uint32_t xvalid[NPC];
#pragma unroll
    for (int m = 0; m < NPC; ++m) {
        const unsigned p = (unsigned)(px_tile * BPX + 32 * m + cp);
        const bool ok = p < (unsigned)S.P;
        const unsigned pn = ok ? p / (unsigned)hw : 0u;
        const unsigned prem = ok ? p - pn * (unsigned)hw : 0u;
        const int oh = (int)(prem / (unsigned)S.wo), ow = (int)prem - oh * S.wo;
        const int ih0 = oh * A.stride - A.pad, iw0 = ow * A.stride - A.pad;
        // (ih0 > -kh and iw0 > -kw: pad < kh, kw)
        const uint32_t rows = ((1u << min(max(S.h - ih0, 0), A.kh)) - 1) & ~((1u << max(-ih0, 0)) - 1);
        const uint32_t cols = ((1u << min(max(S.w - iw0, 0), A.kw)) - 1) & ~((1u << max(-iw0, 0)) - 1);
        xvalid[m] = ok ? rows | cols << 16 : 0u;
        xbase[m] = (((int)pn * S.h + ih0) * S.w + iw0) * row_bytes;
    }
    const buf_rsrc xr = make_rsrc(S.x, S.n * S.h * S.w * row_bytes);
    // this lane's chunk of the stage being loaded: tap (tr, tq), chunk cc of the
    // tap; a tap past the window's last row finds no valid bit
    const int cpt = A.cin / 32;
    int cc, tq, tr;
    {
        const int tap = c8 / cpt;
        cc = c8 - tap * cpt;
        tr = tap / A.kw;
        tq = tap - tr * A.kw;
    }
    int x_off = 0;
    uint32_t x_need = 0;
    auto set_copy = [&]() {
        x_off = (tr * S.w + tq) * row_bytes + XB * cc;
        x_need = tr < 15 ? (1u << tr) | (1u << (16 + tq)) : 0xFFFFFFFFu;
    };
    set_copy();
    auto advance = [&]() {
        auto wrap = [&]() {
            const bool over = cc >= cpt;
            cc -= over ? cpt : 0;
            tq += over ? 1 : 0;
            const bool row = tq == A.kw;
            tq = row ? 0 : tq;
            tr += row ? 1 : 0;
        };
        cc += 8;
        wrap();
        if (cpt < 8)   // a stage spans several taps
            for (int t = cpt; t < 8; t += cpt)
                wrap();
        tr = min(tr, 15);
        set_copy();
    };
    using piece_t = typename std::conditional<F6, v4i, uint2>::type;
    auto load_piece = [&](int m) -> piece_t {
        const int off = (xvalid[m] & x_need) == x_need ? xbase[m] + x_off : (int)0x80000000;
        if constexpr (F6)
            return load_b128(xr, off, 0);
        else
            return load_b64(xr, off, 0);
    };
    // LDS: 16-byte column c of pixel p at 128 p + 16 (c ^ (p & 7)); e2m3: 8-byte
    // column c at Y + 64 p + 8 (c ^ ((p >> 1) & 7))
    const uint32_t wx = XROW * cp + 16 * (c8 ^ (cp & 7));
    const uint32_t wy = BPX * XROW + YROW * cp + 8 * (c8 ^ ((cp >> 1) & 7));
    auto write_piece = [&](uint32_t buf, int m, const piece_t v) {
        if constexpr (F6) {
            const v8i o = spread_e2m3(v);
            *(v4i *)(lds + buf + m * (32 * XROW) + wx) = v4i{o[0], o[1], o[2], o[3]};
            *(uint2 *)(lds + buf + m * (32 * YROW) + wy) = make_uint2((uint32_t)o[4], (uint32_t)o[5]);
        } else {
            const v8i o = spread_e2m1(v);
            *(v4i *)(lds + buf + m * (32 * XROW) + wx) = v4i{o[0], o[1], o[2], o[3]};
        }
    };
    // fragment of K step q of a stage, column tile j of this wave: pixel
    // 16 (NJ wp + j) + r, chunk 4q + g
    const int pw = 16 * NJ * wp + r;
    struct Frag {
        v4i x;
        uint2 y;
    };
    const uint32_t fx0 = XROW * pw + 16 * (g ^ (r & 7)), fx1 = XROW * pw + 16 * ((4 + g) ^ (r & 7));
    const uint32_t fy0 = BPX * XROW + YROW * pw + 8 * (g ^ ((r >> 1) & 7)),
                   fy1 = BPX * XROW + YROW * pw + 8 * ((4 + g) ^ ((r >> 1) & 7));
    auto read_frag = [&](uint32_t buf, int q, int j) -> Frag {
        Frag f;
        f.x = *(const v4i *)(lds + buf + (q ? fx1 : fx0) + j * (16 * XROW));
        f.y = make_uint2(0, 0);
        if constexpr (F6)
            f.y = *(const uint2 *)(lds + buf + (q ? fy1 : fy0) + j * (16 * YROW));
        return f;
    };

    // ---- weights of this wave's 64-channel group (a group past the last reads
    // zeros: the resource then has no bytes)
    const int ct = co_tile * WC + wc;
    const int groups = A.cout_pad / 64;
    const buf_rsrc wr = make_rsrc(S.wt + (long long)ct * KS * (4 * WB), ct < groups ? KS * (4 * WB) : 0);
    struct Wt {
        v4i x;
        uint2 y;
    };
    auto load_w = [&](int k, int i) -> Wt {
        Wt w;
        const int ko = min(k, KS) * (4 * WB) + i * WB;   // a step past the last: past the buffer's end
        w.x = load_b128(wr, lane * 16, ko);
        w.y = make_uint2(0, 0);
        if constexpr (F6)
            w.y = load_b64(wr, lane * 8, ko + 1024);
        return w;
    };

    v4f acc[MI][NJ];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
            acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};

    // ---- prologue: stage 0 in LDS, the first half of stage 1's pieces in
    // registers, weights of step 0
    piece_t rb[PPS];
    Wt fa[2][MI];
    {
        piece_t r0[NPC];
#pragma unroll
        for (int m = 0; m < NPC; ++m)
            r0[m] = load_piece(m);
#pragma unroll
        for (int i = 0; i < MI; ++i)
            fa[0][i] = load_w(0, i);
        advance();   // copy state: stage 1
#pragma unroll
        for (int m = 0; m < PPS; ++m)
            rb[m] = load_piece(m);
#pragma unroll
        for (int m = 0; m < NPC; ++m)
            write_piece(0, m, r0[m]);
    }
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    Frag fb[NJ];
#pragma unroll
    for (int j = 0; j < RA; ++j)
        fb[j] = read_frag(0, 0, j);

    // ---- main loop, one stage per pass. During stage t (buffer t % 2) the
    // pieces of stage t + 1 are widened into the other buffer: their first half
    // in the first step, each before the load of a piece of the second half into
    // its registers, the second half in the second step, each before the load of
    // a first-half piece of stage t + 2. The weights of step k + 1 are loaded
    // during the first column tiles of step k. The barrier in the second step,
    // before the first read of stage t + 1, makes that stage visible; every read
    // of stage t - 1 came before the barrier of stage t - 1.
    uint32_t buf = 0;
    for (int t = 0; t < NST; ++t) {
        static_for<2>([&](auto qc) {
            constexpr int q = decltype(qc)::value;
            static_for<NJ>([&](auto jc) {
                constexpr int j = decltype(jc)::value;
                if constexpr (q == 1 && j == NJ - RA)
                    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
                if constexpr (j < 2) {
                    fa[q ^ 1][2 * j] = load_w(2 * t + q + 1, 2 * j);
                    fa[q ^ 1][2 * j + 1] = load_w(2 * t + q + 1, 2 * j + 1);
                }
                if constexpr (j + RA < NJ)
                    fb[j + RA] = read_frag(buf, q, j + RA);
                else
                    fb[j + RA - NJ] = read_frag(q == 0 ? buf : buf ^ STAGE, q ^ 1, j + RA - NJ);
                // one piece in every second column tile from the third on
                constexpr int pj = NJ >= 8 ? (j >= 2 && j % 2 == 0 ? (j - 2) / 2 : -1) : j < 2 ? j : -1;
                if constexpr (pj >= 0 && pj < PPS) {
                    if constexpr (q * PPS + pj < NPC)
                        write_piece(buf ^ STAGE, q * PPS + pj, rb[pj]);
                    if constexpr ((q ^ 1) * PPS + pj < NPC)
                        rb[pj] = load_piece((q ^ 1) * PPS + pj);
                }
                const v8i b = v8i{fb[j].x.x, fb[j].x.y, fb[j].x.z, fb[j].x.w, (int)fb[j].y.x, (int)fb[j].y.y, 0, 0};
#pragma unroll
                for (int i = 0; i < MI; ++i) {
                    const Wt &w = fa[q][i];
                    acc[i][j] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(
                        v8i{w.x.x, w.x.y, w.x.z, w.x.w, (int)w.y.x, (int)w.y.y, 0, 0}, b, acc[i][j],
                        F6 ? 2 : 4, F6 ? 2 : 4, 0, 0, 0, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
            });
            if constexpr (q == 0)
                advance();
        });
        buf ^= STAGE;
    }

    fx_epilogue<KIND, WC, NJ, OUTK, SKK, FAST>(A, S, lds, ftab, acc, co_tile, tid, [&](int p) -> long long {
        const long long px = (long long)px_tile * BPX + p;
        return px < S.P ? px : -1;
    });
}

// 3x3, stride 1, pad 1 convolutions with the input tile kept in LDS for all nine
// taps: a block of 32 CB input channels of every pixel that the tile's windows
// touch is widened into LDS once, and the K steps of the nine taps then run with
// neither copies nor barriers, reading their fragments at shifted pixels (the
// tiled kernel above widens each pixel up to nine times, and waits once per stage).
//
// The tile's BPX pixels are consecutive in a virtual image that stands in for the
// padding: rows of W + 1 (the extra pixel is the right pad of its row and the left
// pad of the next), H + 1 rows per image (the extra row is the bottom pad of its
// image and the top pad of the next). A window then is three runs of BPX + 2
// consecutive virtual pixels, W + 1 apart, whatever rows and images it spans, and a
// tile loses only the virtual pixels it holds (2% at 100 x 167).
//
// 3x3 256 -> 256 on 267200 pixels: 107 us on the kernel above, 94 here (140 on the
// int8 kernel); 128 -> 128 on 133600: 30.5 -> 21.2; 2 bits 21.6 -> 18.1.
//
// Weights one K step ahead in registers, activation fragments RA column tiles
// ahead. Input channels beyond a block (256, or 128 for layers of 128): block after
// block, two barriers each.
// MULTI: more than one block (else cin is the block's)
template <int KIND, int WC, int NJ, int OUTK, int SKK, int FAST, int CB, int MULTI>
__global__ void __launch_bounds__(256, 2) qconv_fx3_kernel(MfmaArgs A)
{
    constexpr bool F6 = KIND == GF_F6;
    constexpr int WP = 4 / WC, MI = 4;
    constexpr int Q = CB == 8 ? 2 : 1;               // K steps per tap and block (CB 2: per pair of taps)
    constexpr int BPX = 16 * NJ * WP, RUN = BPX + 2, NPX = 3 * RUN;
    constexpr int XB = F6 ? 16 : 8;                  // packed bytes of a chunk
    constexpr int WB = F6 ? GF_F6_TILE : 1024;       // weight bytes of a row tile and K step
    constexpr int XROW = 16 * CB, YROW = F6 ? 8 * CB : 0;
    constexpr int TAB = (NPX * 4 + 127) / 128 * 128;
    constexpr int DATA = NPX * (XROW + YROW);
    constexpr int EPIB = fx_epilogue_bytes<KIND, WC, NJ, OUTK, SKK>();
    constexpr bool EARLY = FAST == 2 && SKK == 0 && OUTK == 0;
    constexpr int OFF_F = TAB + (DATA > EPIB ? (DATA + 15) / 16 * 16 : EPIB);
    constexpr int LDS = OFF_F + (EARLY ? 2 * WC * 256 : 0);
    constexpr int PPI = 256 / CB, IT = (NPX + PPI - 1) / PPI;   // pixels per copy pass, passes
    constexpr int RA = NJ >= 8 ? 2 : 1;
    static_assert(CB == 8 || CB == 4 || CB == 2, "chunks per block");
    static_assert(CB == 8 || !MULTI, "blocks of 8 chunks");
    __shared__ __attribute__((aligned(1024))) uint8_t lds[LDS];
    int *const tab = (int *)lds;                     // input pixel of virtual pixel i of run t, or -1
    uint8_t *const data = lds + TAB;

    const int bid = blockIdx.x;
    const int tile = (bid & 7) * A.tiles_per_xcd + (bid >> 3);
    if (tile >= A.total_tiles)
        return;
    int s = 0;
    if (A.nseg > 1) {
#pragma unroll
        for (int i = 1; i < AQD_MAX_SEGS; ++i)
            if (i < A.nseg && tile >= A.seg[i].tile_begin)
                s = i;
    }
    const MfmaSeg &S = A.seg[s];
    const int t_in_seg = tile - S.tile_begin;
    const int co_tile = t_in_seg % A.co_tiles;
    const int px_tile = t_in_seg / A.co_tiles;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wc = wave % WC, wp = wave / WC;
    const int r = lane & 15, g = lane >> 4;
    const int32_t *const ftab = (const int32_t *)(lds + OFF_F % LDS);
    if constexpr (EARLY)
        fx_early_table<WC>(A, S, ftab, co_tile, tid);
    const int KS = A.ksteps, kpt = CB == 2 ? 1 : A.cin / 128;   // K steps, per tap
    const int nblk = MULTI ? A.cin / (32 * CB) : 1;
    const int row_bytes = A.cin * XB / 32;

    // ---- weights of this wave's 64-channel group (as in the kernel above)
    const int ct = co_tile * WC + wc;
    const buf_rsrc wr = make_rsrc(S.wt + (long long)ct * KS * (4 * WB), ct < A.cout_pad / 64 ? KS * (4 * WB) : 0);
    struct Wt {
        v4i x;
        uint2 y;
    };
    auto load_w = [&](int k, int i) -> Wt {
        Wt w;
        const int ko = k * (4 * WB) + i * WB;
        w.x = load_b128(wr, lane * 16, ko);
        w.y = make_uint2(0, 0);
        if constexpr (F6)
            w.y = load_b64(wr, lane * 8, ko + 1024);
        return w;
    };
    // the K step of tap (ty, tx), step q of block blk, in the stored order (tap,
    // then channel)
    auto kidx = [&](int blk, int ty, int tx, int q) -> int { return (3 * ty + tx) * kpt + blk * Q + q; };

    // ---- the virtual pixels of the three runs
    const int vw = S.w + 1, vh = S.h + 1;
    for (int p = tid; p < NPX; p += 256) {
        const int t = p / RUN, i = p - t * RUN;
        const int v = px_tile * BPX - 1 + i + (t - 1) * vw;
        int at = -1;
        if (v >= 0) {
            const unsigned vy = (unsigned)v / (unsigned)vw, x = (unsigned)v - vy * (unsigned)vw;
            const unsigned n = vy / (unsigned)vh, y = vy - n * (unsigned)vh;
            if (x < (unsigned)S.w && y < (unsigned)S.h && n < (unsigned)S.n)
                at = (int)((n * (unsigned)S.h + y) * (unsigned)S.w + x);
        }
        tab[p] = at;
    }
    __syncthreads();

    const buf_rsrc xr = make_rsrc(S.x, S.n * S.h * S.w * row_bytes);
    const int cc = tid % CB, cp0 = tid / CB;
    using piece_t = typename std::conditional<F6, v4i, uint2>::type;
    // LDS column c of the row of virtual pixel i of a run (16-byte columns, then the
    // 8-byte ones): XOR with i, so that 16 consecutive pixels at one column fall on
    // all banks
    auto xcol = [](int i, int c) -> int {
        return CB == 8 ? c ^ (i & 7) : CB == 4 ? c ^ ((i >> 1) & 3) : c ^ ((i >> 2) & 1);
    };
    auto ycol = [](int i, int c) -> int {
        return CB == 8 ? c ^ ((i >> 1) & 7) : CB == 4 ? c ^ ((i >> 2) & 3) : c ^ ((i >> 3) & 1);
    };
    // copy passes it0 .. it0 + n of a block: loads, then widening and LDS writes
    auto stage = [&](int blk, int cp, auto it0c, auto nc) {
        constexpr int it0 = decltype(it0c)::value, n = decltype(nc)::value;
        piece_t v[n];
#pragma unroll
        for (int k = 0; k < n; ++k) {
            const int p = (it0 + k) * PPI + cp;
            const int at = p < NPX ? tab[p] : -1;
            const int off = at >= 0 ? at * row_bytes + blk * (XB * CB) + XB * cc : (int)0x80000000;
            if constexpr (F6)
                v[k] = load_b128(xr, off, 0);
            else
                v[k] = load_b64(xr, off, 0);
        }
#pragma unroll
        for (int k = 0; k < n; ++k) {
            const int p = (it0 + k) * PPI + cp;
            if (it0 + k == IT - 1 && p >= NPX)
                continue;
            const int i = p - (p >= RUN ? RUN : 0) - (p >= 2 * RUN ? RUN : 0);
            uint8_t *x = data + p * XROW + 16 * xcol(i, cc);
            if constexpr (F6) {
                const v8i o = spread_e2m3(v[k]);
                *(v4i *)x = v4i{o[0], o[1], o[2], o[3]};
                *(uint2 *)(data + NPX * XROW + p * YROW + 8 * ycol(i, cc)) = make_uint2((uint32_t)o[4], (uint32_t)o[5]);
            } else {
                const v8i o = spread_e2m1(v[k]);
                *(v4i *)x = v4i{o[0], o[1], o[2], o[3]};
            }
        }
    };
    // the first block: every load in flight at once (nothing else holds registers)
    stage(0, cp0, std::integral_constant<int, 0>{}, std::integral_constant<int, IT>{});
    Wt fa[2][MI];
#pragma unroll
    for (int i = 0; i < MI; ++i)
        fa[0][i] = load_w(0, i);
    __syncthreads();

    // ---- fragments: column tile j of tap (ty, tx), step q: virtual pixel
    // 16 (NJ wp + j) + r + tx of run ty, chunk 4q + g
    struct Frag {
        v4i x;
        uint2 y;
    };
    // (CB 2: a step holds two taps, lane groups 0-1 the first and 2-3 the second;
    // ax[k], ay[k] are those of step k of the five, the last tap of the last step is
    // past the window and meets zero weights)
    constexpr int NA = CB == 2 ? 5 : 3;
    uint32_t ax[NA], ay[NA];
#pragma unroll
    for (int k = 0; k < NA; ++k) {
        const int tap = CB == 2 ? min(2 * k + (g >> 1), 8) : k;   // CB > 2: tap k of row 0
        const int c = CB == 2 ? g & 1 : g;
        const int run = tap / 3, i = 16 * NJ * wp + r + tap - 3 * run;
        ax[k] = (uint32_t)(XROW * (run * RUN + i) + 16 * xcol(i, c));
        ay[k] = (uint32_t)(NPX * XROW + YROW * (run * RUN + i) + 8 * ycol(i, c));
    }
    // (ax and ay move to window row ty0 with the loop below; rows: from there)
    auto read_frag = [&](int rows, int tx, int q, int j) -> Frag {
        Frag f;
        // chunk 4 + g: bit 2 of the column flips
        f.x = *(const v4i *)(data + (q ? ax[tx] ^ 64u : ax[tx]) + (rows * RUN + 16 * j) * XROW);
        f.y = make_uint2(0, 0);
        if constexpr (F6)
            f.y = *(const uint2 *)(data + (q ? ay[tx] ^ 32u : ay[tx]) + (rows * RUN + 16 * j) * YROW);
        return f;
    };

    v4f acc[MI][NJ];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
            acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
    Frag fb[NJ];
    for (int blk = 0; blk < nblk; ++blk) {
        if (MULTI && blk) {
            __syncthreads();   // every wave is done with the last block
            int cp = cp0;
            asm volatile("" : "+v"(cp));   // (addresses worked out here, not kept through the K loop)
            static_for<(IT + 3) / 4>([&](auto bc) {
                constexpr int it0 = 4 * decltype(bc)::value;
                stage(blk, cp, std::integral_constant<int, it0>{}, std::integral_constant<int, (IT - it0 < 4 ? IT - it0 : 4)>{});
            });
            __syncthreads();
        }
#pragma unroll
        for (int j = 0; j < RA; ++j)
            fb[j] = read_frag(0, 0, 0, j);
        // window rows; with one K step per tap (odd counts per row) all nine taps
        // are one body, so that the weight sets stay compile-time
        constexpr int TYU = Q == 1 ? 3 : 1, U = CB == 2 ? 5 : 3 * Q * TYU;
        for (int ty0 = 0; ty0 < 3; ty0 += TYU) {
            static_for<U>([&](auto uc) {
                constexpr int u = decltype(uc)::value;
                constexpr int un = u + 1 < U ? u + 1 : 0;
                constexpr int tx = CB == 2 ? u : u / Q % 3, q = u % Q;
                constexpr int txn = CB == 2 ? un : un / Q % 3, qn = un % Q;
                constexpr int row = CB == 2 ? 0 : u / (3 * Q);
                // the next step; after the block's last: the next block's first
                // (after the last block's: read, not used)
                const int rown = CB == 2 ? 0 : u + 1 < U ? (u + 1) / (3 * Q) : ty0 + TYU < 3 ? TYU : -ty0;
                const int bn = u + 1 < U || ty0 + TYU < 3 ? blk : blk + 1;
                const int kn = bn < nblk ? kidx(bn, CB == 2 ? 0 : ty0 + rown, txn, qn) : 0;
                static_for<NJ>([&](auto jc) {
                    constexpr int j = decltype(jc)::value;
                    if constexpr (j < 2) {
                        fa[(u + 1) % 2][2 * j] = load_w(kn, 2 * j);
                        fa[(u + 1) % 2][2 * j + 1] = load_w(kn, 2 * j + 1);
                    }
                    if constexpr (j + RA < NJ)
                        fb[j + RA] = read_frag(row, tx, q, j + RA);
                    else
                        fb[j + RA - NJ] = read_frag(rown, txn, qn, j + RA - NJ);
                    const v8i b = v8i{fb[j].x.x, fb[j].x.y, fb[j].x.z, fb[j].x.w, (int)fb[j].y.x, (int)fb[j].y.y, 0, 0};
#pragma unroll
                    for (int i = 0; i < MI; ++i) {
                        const Wt &w = fa[u % 2][i];
                        acc[i][j] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(
                            v8i{w.x.x, w.x.y, w.x.z, w.x.w, (int)w.y.x, (int)w.y.y, 0, 0}, b, acc[i][j],
                            F6 ? 2 : 4, F6 ? 2 : 4, 0, 0, 0, 0);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                });
            });
            const int d = ty0 + TYU < 3 ? TYU : -ty0;
#pragma unroll
            for (int tx = 0; tx < (CB == 2 ? 0 : 3); ++tx) {
                ax[tx] += (uint32_t)(d * (RUN * XROW));
                ay[tx] += (uint32_t)(d * (RUN * YROW));
            }
        }
    }
    // (the thread's number from its lane, so that none is held through the K loop)
    const int tid2 = 64 * wave + (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    fx_epilogue<KIND, WC, NJ, OUTK, SKK, FAST>(A, S, data, ftab, acc, co_tile, tid2, [&](int p) -> long long {
        return tab[RUN + 1 + p];
    });
}

template <int KIND, int WC, int NJ>
hipError_t launch_modes(const MfmaArgs &a, int fast, hipStream_t stream)
{
    const dim3 grid(8 * a.tiles_per_xcd), block(256);
    // workgroups per CU: what the registers allow without spilling
    constexpr int OCC = NJ == 4 && KIND == GF_F4 ? 3 : 2;
    if (a.bits_out == 32)
        hipLaunchKernelGGL((qconv_fx_kernel<KIND, WC, NJ, 1, 0, 1, 2>), grid, block, 0, stream, a);
    else if (a.skip_bits == 0 && fast == 2)
        hipLaunchKernelGGL((qconv_fx_kernel<KIND, WC, NJ, 0, 0, 2, OCC>), grid, block, 0, stream, a);
    else if (a.skip_bits == 0 && fast)
        hipLaunchKernelGGL((qconv_fx_kernel<KIND, WC, NJ, 0, 0, 1, OCC>), grid, block, 0, stream, a);
    else if (a.skip_bits == 0)
        hipLaunchKernelGGL((qconv_fx_kernel<KIND, WC, NJ, 0, 0, 0, 2>), grid, block, 0, stream, a);
    else if constexpr (NJ == 8 && KIND == GF_F6)
        return hipErrorInvalidValue;   // the skip codes do not fit beside 128 accumulators
    else if (fast == 2)
        hipLaunchKernelGGL((qconv_fx_kernel<KIND, WC, NJ, 0, 1, 2, 2>), grid, block, 0, stream, a);
    else if (fast)
        hipLaunchKernelGGL((qconv_fx_kernel<KIND, WC, NJ, 0, 1, 1, 2>), grid, block, 0, stream, a);
    else
        hipLaunchKernelGGL((qconv_fx_kernel<KIND, WC, NJ, 0, 1, 0, 2>), grid, block, 0, stream, a);
    return hipGetLastError();
}

template <int KIND, int WC, int NJ, int CB, int MULTI>
hipError_t launch3_modes(const MfmaArgs &a, int fast, hipStream_t stream)
{
    const dim3 grid(8 * a.tiles_per_xcd), block(256);
    if (a.bits_out == 32)
        hipLaunchKernelGGL((qconv_fx3_kernel<KIND, WC, NJ, 1, 0, 1, CB, MULTI>), grid, block, 0, stream, a);
    else if (a.skip_bits == 0 && fast == 2)
        hipLaunchKernelGGL((qconv_fx3_kernel<KIND, WC, NJ, 0, 0, 2, CB, MULTI>), grid, block, 0, stream, a);
    else if (a.skip_bits == 0 && fast)
        hipLaunchKernelGGL((qconv_fx3_kernel<KIND, WC, NJ, 0, 0, 1, CB, MULTI>), grid, block, 0, stream, a);
    else if (a.skip_bits == 0)
        hipLaunchKernelGGL((qconv_fx3_kernel<KIND, WC, NJ, 0, 0, 0, CB, MULTI>), grid, block, 0, stream, a);
    else if constexpr (NJ == 8)
        return hipErrorInvalidValue;   // (as above: no room for the skip codes)
    else if (fast == 2)
        hipLaunchKernelGGL((qconv_fx3_kernel<KIND, WC, NJ, 0, 1, 2, CB, MULTI>), grid, block, 0, stream, a);
    else if (fast)
        hipLaunchKernelGGL((qconv_fx3_kernel<KIND, WC, NJ, 0, 1, 1, CB, MULTI>), grid, block, 0, stream, a);
    else
        hipLaunchKernelGGL((qconv_fx3_kernel<KIND, WC, NJ, 0, 1, 0, CB, MULTI>), grid, block, 0, stream, a);
    return hipGetLastError();
}

template <int KIND>
hipError_t launch_kind(const MfmaArgs &a, const GfPlan &p, int fast, hipStream_t stream)
{
    if (p.kw < 0) {   // 3x3, stride 1: the input tile in LDS
        const int tile = p.mi * 10 + p.nj;
        if (a.cin == 256)
            return tile == 48   ? launch3_modes<KIND, 4, 8, 8, 0>(a, fast, stream)
                   : tile == 44 ? launch3_modes<KIND, 4, 4, 8, 0>(a, fast, stream)
                   : tile == 24 ? launch3_modes<KIND, 2, 4, 8, 0>(a, fast, stream)
                                : hipErrorInvalidValue;
        if (a.cin == 128)
            return tile == 24 ? launch3_modes<KIND, 2, 4, 4, 0>(a, fast, stream) : hipErrorInvalidValue;
        if (a.cin == 64)
            return tile == 14 ? launch3_modes<KIND, 1, 4, 2, 0>(a, fast, stream) : hipErrorInvalidValue;
        return tile == 44 ? launch3_modes<KIND, 4, 4, 8, 1>(a, fast, stream) : hipErrorInvalidValue;
    }
    switch (p.mi * 10 + p.nj) {   // waves along channels, column tiles per wave
    case 48: return launch_modes<KIND, 4, 8>(a, fast, stream);
    case 44: return launch_modes<KIND, 4, 4>(a, fast, stream);
    case 24: return launch_modes<KIND, 2, 4>(a, fast, stream);
    }
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_qconv_fx(const MfmaArgs &a, const GfPlan &p, hipStream_t stream)
{
    const bool f6 = p.kind == GF_F6;
    if ((p.kind != GF_F6 && p.kind != GF_F4) || a.ksplit != 1 || a.part != 0 || a.kh > 7 || a.kw > 7 ||
        a.cin % 32 != 0 || a.ksteps != (a.kh * a.kw * (a.cin / 32) + 3) / 4 || a.cout_pad % 64 != 0 ||
        a.cout > a.cout_pad || a.co_tiles != (a.cout_pad / 64 + p.mi - 1) / p.mi ||
        (a.bits_out == 32 ? a.cout % 4 != 0 || a.skip_bits != 0
                          : a.cout % 16 != 0 || a.bits_out != (f6 ? 4 : 2) ||
                                (a.skip_bits != 0 && a.skip_bits != a.bits_out)) ||
        (long long)a.ksteps * 4 * (f6 ? GF_F6_TILE : 1024) >= (1LL << 31))
        return hipErrorInvalidValue;
    if (p.kw < 0 && (a.kh != 3 || a.kw != 3 || a.stride != 1 || a.pad != 1 || (a.cin % 256 != 0 && a.cin != 128 && a.cin != 64)))
        return hipErrorInvalidValue;
    // 32-bit buffer offsets and pixel numbers (virtual pixels: at most 4 per pixel)
    for (int i = 0; i < a.nseg; ++i)
        if ((p.kw < 0 && (long long)a.seg[i].n * (a.seg[i].h + 1) * (a.seg[i].w + 1) + 512 >= (1LL << 31)) ||
            (long long)a.seg[i].n * a.seg[i].h * a.seg[i].w * a.cin / (f6 ? 2 : 4) >= (1LL << 31) ||
            a.seg[i].P + 256 >= (1LL << 31))
            return hipErrorInvalidValue;
    int fast = 2;
    for (int i = 0; i < a.nseg; ++i)
        fast = a.seg[i].fast < fast ? a.seg[i].fast : fast;
    return f6 ? launch_kind<GF_F6>(a, p, fast, stream) : launch_kind<GF_F4>(a, p, fast, stream);
}

}  // namespace aqd
