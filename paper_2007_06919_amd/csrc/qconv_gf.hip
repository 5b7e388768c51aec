// Global-fed implicit-GEMM integer convolution: every wave reads both operands
// from global memory (L1/L2) straight into registers, no LDS and no barrier in
// its K loop, and the waves of a workgroup split the K range between them and
// add their sums through LDS at the end. For launches too small to fill the GPU
// (one image, the coarse pyramid levels, small layers) and for shapes the tiled
// kernels do not take (1 to 3 output channels, 8-bit codes in and out, input
// channels that are only a multiple of 32).
//
// What bounds such a launch is the length of its serial chain: a tile's K steps
// run one after another on one wave's MFMAs at the latency of a copy, a barrier
// and an LDS read each, with most of the chip idle. Here a tile is 64 x 64 or
// smaller, its K range is cut between 1 to 4 waves, each wave keeps the loads of
// three or four steps in flight, and the sums are combined inside the workgroup
// (no second launch, no partial sums in memory). 3x3 256 -> 256 on 4200 pixels:
// 27.6 -> 11.3 us, 3x3 64 -> 64 on 1024: 14.9 -> 4.6 us (more at the rule that
// picks it, plan_gf). What is left there is the launch (about 4 us on a tiny
// layer) and, at several hundred tiles, the L1's delivery of both operands to
// every wave: 13 to 26 bytes per clock and CU.
//
// Operands (Eq. 4, Sec. 3.2.1: rows = output channels, columns = pixels, K =
// taps x input channels; a K step is four chunks of one tap's consecutive
// channels, one chunk per lane group; a step may span taps):
//  * F6: codes of 2..4 bits stored in 4-bit containers with weights of at most
//    4 bits on v_mfma_f32_16x16x128_f8f6f4, both operands e2m3 (32 channels per
//    chunk). e2m3 holds k / 8 for every integer |k| <= 15, with the bit pattern
//    of k itself (subnormal below 8), so widening 4-bit codes is moving them to
//    6-bit fields. Twice the rate of the int8 MFMA.
//  * F4: 2-bit codes with 2-bit weights on the same MFMA, both e2m1 (a code k
//    reads as k / 2; the weights are exact).
//  * I8: 8-bit codes re-centred by -128 on v_mfma_i32_16x16x64_i8 (16 channels
//    per chunk); the bias carries 128 * sum(w).
// Exactness of the float kinds: products are integers times 2^-6 (F6) or 2^-1
// (F4), and every partial sum is below 2^24 of these units (checked at create:
// K * max code * max |w| < 2^24), so fp32 holds each sum exactly in any order.
//
// Epilogue (Sec. 3.2.2-3.2.3, Eq. 6-8, Eq. 2 on integers): each wave finishes
// its share of the tile's accumulators; a lane holds 4 * IG consecutive channels
// of one pixel. Output and skip widths and the 32- or 64-bit requantisation are
// uniform run-time choices: a lane finishes at most 64 values.

#include "epilogue.h"
#include "internal.h"
#include "mfma_common.h"

namespace aqd {
namespace {

typedef float v4f __attribute__((ext_vector_type(4)));

constexpr int GF_TAB = EPI_FIELDS * 64 * 4;          // LDS bytes of a 64-channel group's tables

// EP: 0 = int32 outputs, 1 = codes, 2 = codes with a skip
template <int KIND, int MI, int NJ, int KW, int EP>
__global__ void __launch_bounds__(64 * KW, 2) qconv_gf_kernel(MfmaArgs A)
{
    constexpr bool F6 = KIND == GF_F6, F4 = KIND == GF_F4, I8 = KIND == GF_I8;
    constexpr int XB = F4 ? 8 : 16;                  // activation bytes of a chunk
    constexpr int WB = F6 ? GF_F6_TILE : 1024;       // weight bytes of a 16-row tile and K step
    constexpr int D = MI * NJ >= 16 ? 3 : 4;         // steps in flight per wave
    constexpr int IGU = MI * NJ / KW;                // accumulators a wave finishes
    constexpr int IG = KW <= NJ ? MI : IGU;          // of these, per pixel column (4 channels each)
    constexpr int JU = IGU / IG;                     // pixel columns a wave finishes
    static_assert(MI * NJ % KW == 0 && IG * JU == IGU && MI % IG == 0, "the tile splits over the waves");
    using acc_t = typename std::conditional<I8, v4i, v4f>::type;
    using raw_t = typename std::conditional<F4, uint2, v4i>::type;
    __shared__ __attribute__((aligned(1024))) uint8_t lds[GF_TAB + (KW - 1) * MI * NJ * 1024];
    uint8_t *const red = lds + GF_TAB;               // the waves' sums

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
    // (a workgroup takes MI row tiles of a 64-channel group; co_tiles counts them)
    const int co_tile = t_in_seg % A.co_tiles;
    const int px_tile = t_in_seg / A.co_tiles;
    const int ct = co_tile / (4 / MI), i0 = (co_tile % (4 / MI)) * MI;

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = lane & 15, g = lane >> 4;
    // the group's epilogue tables: copied to LDS while the K loop runs
    if (wave == 0) {
        const int32_t *src = S.epi + 64 * ct + (lane >> 4) * A.cout_pad + 4 * (lane & 15);
        dma16(src, lds_addr(lds));
        dma16(src + 4 * A.cout_pad, lds_addr(lds) + GF_TAB / 2);
    }
    const int hw = S.ho * S.wo;
    const int KS = A.ksteps;
    const int s0 = KS * wave / KW, s1 = KS * (wave + 1) / KW;   // this wave's K steps

    // ---- pixels: byte offset of the window's origin, and which window rows
    // (bit t) and columns (bit 16 + t) lie inside the image (none past the
    // end); lane l works them out for pixel l of the tile, the lanes of column
    // tile j then fetch theirs
    const int row_bytes = I8 ? A.cin : F4 ? A.cin / 4 : A.cin / 2;
    int xbase[NJ];
    uint32_t xvalid[NJ];
    {
        const unsigned p = (unsigned)(px_tile * (16 * NJ) + lane % (16 * NJ));
        const bool ok = p < (unsigned)S.P;
        const unsigned pn = ok ? p / (unsigned)hw : 0u;
        const unsigned prem = ok ? p - pn * (unsigned)hw : 0u;
        const int oh = (int)(prem / (unsigned)S.wo), ow = (int)prem - oh * S.wo;
        const int ih0 = oh * A.stride - A.pad, iw0 = ow * A.stride - A.pad;
        // (ih0 > -kh and iw0 > -kw: pad < kh, kw)
        const uint32_t rows = ((1u << min(max(S.h - ih0, 0), A.kh)) - 1) & ~((1u << max(-ih0, 0)) - 1);
        const uint32_t cols = ((1u << min(max(S.w - iw0, 0), A.kw)) - 1) & ~((1u << max(-iw0, 0)) - 1);
        const uint32_t v = ok ? rows | cols << 16 : 0u;
        const int base = (((int)pn * S.h + ih0) * S.w + iw0) * row_bytes;
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            xvalid[j] = (uint32_t)__shfl((int)v, 16 * j + r);
            xbase[j] = __shfl(base, 16 * j + r);
        }
    }
    const buf_rsrc xr = make_rsrc(S.x, S.n * S.h * S.w * row_bytes);
    const buf_rsrc wr = make_rsrc(S.wt + ((long long)ct * KS * 4 + i0) * WB, (KS * 4 - i0) * WB);

    // this lane group's chunk of the step being loaded: tap (tr, tq), chunk cc
    // of the tap; a tap past the window's last row finds no valid bit
    const int cpt = A.cin / (I8 ? 16 : 32);          // chunks per tap
    int cc, tq, tr;
    {
        const int kc = 4 * s0 + g, tap = kc / cpt;
        cc = kc - tap * cpt;
        tr = tap / A.kw;
        tq = tap - tr * A.kw;
    }
    struct Set {
        v4i a[MI];
        uint2 a2[F6 ? MI : 1];
        raw_t b[NJ];
    };
    // (steps past this wave's range load nothing: every offset is past the end)
    auto load_step = [&](int k, Set &q) {
        const bool in = k < s1;
        const int off = (tr * S.w + tq) * row_bytes + XB * cc;
        const uint32_t need = in ? (1u << tr) | (1u << (16 + tq)) : 0xFFFFFFFFu;
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const int o = (xvalid[j] & need) == need ? xbase[j] + off : (int)0x80000000;
            if constexpr (F4)
                q.b[j] = load_b64(xr, o, 0);
            else
                q.b[j] = load_b128(xr, o, 0);
        }
        const int ko = in ? k * (4 * WB) : 0;
        const int l16 = in ? lane * 16 : (int)0x80000000, l8 = in ? lane * 8 : (int)0x80000000;
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            q.a[i] = load_b128(wr, l16 + i * WB, ko);
            if constexpr (F6)
                q.a2[i] = load_b64(wr, l8 + i * WB + 1024, ko);
        }
        cc += 4;
        auto wrap = [&]() {
            const bool over = cc >= cpt;
            cc -= over ? cpt : 0;
            tq += over ? 1 : 0;
            const bool row = tq == A.kw;
            tq = row ? 0 : tq;
            tr += row ? 1 : 0;
        };
        wrap();
        if (cpt < 4)   // a step spans up to four taps
            for (int t = 0; t < 3; ++t)
                wrap();
    };

    acc_t acc[MI][NJ];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
            acc[i][j] = acc_t{0, 0, 0, 0};
    auto mul_step = [&](const Set &q) {
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            if constexpr (I8) {
                const v4i b = q.b[j] ^ v4i{(int)0x80808080, (int)0x80808080, (int)0x80808080, (int)0x80808080};
#pragma unroll
                for (int i = 0; i < MI; ++i)
                    acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(q.a[i], b, acc[i][j], 0, 0, 0);
            } else if constexpr (F4) {
                const v8i b = spread_e2m1(q.b[j]);
#pragma unroll
                for (int i = 0; i < MI; ++i)
                    acc[i][j] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(
                        v8i{q.a[i].x, q.a[i].y, q.a[i].z, q.a[i].w, 0, 0, 0, 0}, b, acc[i][j], 4, 4, 0, 0, 0, 0);
            } else {
                const v8i b = spread_e2m3(q.b[j]);
#pragma unroll
                for (int i = 0; i < MI; ++i)
                    acc[i][j] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(
                        v8i{q.a[i].x, q.a[i].y, q.a[i].z, q.a[i].w, (int)q.a2[i].x, (int)q.a2[i].y, 0, 0}, b,
                        acc[i][j], 2, 2, 0, 0, 0, 0);
            }
        }
    };
    Set set[D];
#pragma unroll
    for (int d = 0; d < D; ++d)
        load_step(s0 + d, set[d]);
    // whole rounds of D steps, each set refilled once it is used; the loads of
    // the last round are past the range
    int k = s0;
    for (; k + D <= s1; k += D)
        static_for<D>([&](auto dc) {
            constexpr int d = decltype(dc)::value;
            mul_step(set[d]);
            load_step(k + d + D, set[d]);
        });
    static_for<D - 1>([&](auto dc) {
        constexpr int d = decltype(dc)::value;
        if (k + d < s1)
            mul_step(set[d]);
    });

    // ---- what this wave finishes, and its skip codes (4 per word), on their
    // way while the waves' sums are exchanged
    const int jw = IGU * wave / MI, iw = IGU * wave % MI;
    const int c0 = 64 * ct + 16 * g + 4 * (i0 + iw);       // first of the lane's 4 * IG channels
    const long long px0 = (long long)px_tile * (16 * NJ) + 16 * jw + r;
    bool ok[JU];
    long long spix[JU];
    uint32_t skw[JU][IG];
#pragma unroll
    for (int jj = 0; jj < JU; ++jj) {
        const long long px = px0 + 16 * jj;
        ok[jj] = px < S.P && c0 < A.cout;
        spix[jj] = px;
#pragma unroll
        for (int q = 0; q < IG; ++q)
            skw[jj][q] = 0;
        if (EP != 2 || !ok[jj])
            continue;
        if (A.up2) {
            const unsigned pn = (unsigned)px / (unsigned)hw, prem = (unsigned)px - pn * (unsigned)hw;
            const unsigned oh = prem / (unsigned)S.wo, ow = prem - oh * (unsigned)S.wo;
            spix[jj] = ((long long)pn * S.hs + (oh >> 1)) * S.ws + (ow >> 1);
        }
        const long long at = spix[jj] * A.cout + c0;       // a multiple of 4 codes
        const uint8_t *sk = (const uint8_t *)S.skip;
        if (IG == 4 && A.skip_bits == 4 && A.cout % 16 == 0) {
            const uint2 t = *(const uint2 *)(sk + at / 2);
            skw[jj][0] = t.x & 0xFFFFu;
            skw[jj][1 % IG] = t.x >> 16;
            skw[jj][2 % IG] = t.y & 0xFFFFu;
            skw[jj][3 % IG] = t.y >> 16;
        } else if (A.skip_bits != 32) {
#pragma unroll
            for (int q = 0; q < IG; ++q)
                if (c0 + 4 * q < A.cout)
                    skw[jj][q] = A.skip_bits == 4   ? (uint32_t)*(const uint16_t *)(sk + at / 2 + 2 * q)
                                 : A.skip_bits == 2 ? (uint32_t)sk[at / 4 + q]
                                                    : *(const uint32_t *)(sk + at + 4 * q);
        }
    }

    // ---- the waves' sums: wave u finishes accumulators IGU * u .. of the
    // column-major order (column j, then row tile i); every other wave's part
    // of them goes through LDS, 16 bytes per lane
    acc_t fin[IGU];
    if constexpr (KW == 1) {
#pragma unroll
        for (int q = 0; q < IGU; ++q)
            fin[q] = acc[q % MI][q / MI];
    } else {
        static_for<KW>([&](auto uc) {
            constexpr int u = decltype(uc)::value;
            if (u == wave) {
#pragma unroll
                for (int q = 0; q < IGU; ++q)
                    fin[q] = acc[(IGU * u + q) % MI][(IGU * u + q) / MI];
            } else {
                const int slot = wave < u ? wave : wave - 1;   // 0 .. KW - 2
#pragma unroll
                for (int q = 0; q < IGU; ++q)
                    *(acc_t *)(red + (((u * (KW - 1) + slot) * IGU + q) * 64 + lane) * 16) =
                        acc[(IGU * u + q) % MI][(IGU * u + q) / MI];
            }
        });
        wait_vmcnt<0>();                                   // the tables' copy
        __syncthreads();
#pragma unroll
        for (int t = 0; t < KW - 1; ++t)
#pragma unroll
            for (int q = 0; q < IGU; ++q)
                fin[q] += *(const acc_t *)(red + (((wave * (KW - 1) + t) * IGU + q) * 64 + lane) * 16);
    }

    // ---------------------------------------------------------------- epilogue
    // fin[IG * jj + q]: row tile i0 + iw + q, pixel column jw + jj of the tile
    constexpr float UNIT = F6 ? 64.f : 2.f;                // float kinds: accumulator units per integer
    if constexpr (KW == 1)
        wait_vmcnt<0>();                                   // the tables' copy
    const int cl = 16 * g + 4 * (i0 + iw);                 // first of the lane's 4 * IG channels, in the group
    const int32_t *tab = (const int32_t *)lds + cl;        // [EPI_FIELDS][64]
    uint32_t word[JU][IG];                                 // 4 output codes each
#pragma unroll
    for (int q = 0; q < IG; ++q) {
        const int c = c0 + 4 * q;
        const v4i bias = *(const v4i *)(tab + 64 * EPI_BIAS + 4 * q);
        int v[JU][4];
#pragma unroll
        for (int jj = 0; jj < JU; ++jj)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if constexpr (I8)   // (int32 all the way: 8-bit sums go past 2^24)
                    v[jj][e] = fin[IG * jj + q][e] + bias[e];
                else
                    v[jj][e] = (int)(fin[IG * jj + q][e] * UNIT) + bias[e];
        if constexpr (EP == 0) {
#pragma unroll
            for (int jj = 0; jj < JU; ++jj) {
                int32_t *y = (int32_t *)S.y + (px0 + 16 * jj) * A.cout + c;
                if (!ok[jj] || c >= A.cout)
                    continue;
                if ((A.cout & 3) == 0) {
                    *(v4i *)y = v4i{v[jj][0], v[jj][1], v[jj][2], v[jj][3]};
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (c + e < A.cout)
                            y[e] = v[jj][e];
                }
            }
            continue;
        }
        // code outputs: cout is a multiple of 4
        v4i sc = {0, 0, 0, 0}, sd = sc, ss = sc;
        if constexpr (EP == 2) {
            sc = *(const v4i *)(tab + 64 * EPI_SKIP_C + 4 * q);
            sd = *(const v4i *)(tab + 64 * EPI_SKIP_D + 4 * q);
            ss = *(const v4i *)(tab + 64 * EPI_SKIP_SIDE + 4 * q);
        }
        const v4i mult = *(const v4i *)(tab + 64 * EPI_MULT + 4 * q);
        const v4i shift = *(const v4i *)(tab + 64 * EPI_SHIFT + 4 * q);
#pragma unroll
        for (int jj = 0; jj < JU; ++jj) {
            int kv[4] = {0, 0, 0, 0};
            if (EP == 2 && A.skip_bits == 32) {
                if (ok[jj] && c < A.cout) {
                    const v4i t = *(const v4i *)((const int32_t *)S.skip + spix[jj] * A.cout + c);
                    kv[0] = t.x; kv[1] = t.y; kv[2] = t.z; kv[3] = t.w;
                }
            } else if constexpr (EP == 2) {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    kv[e] = (int)((skw[jj][q] >> (e * A.skip_bits)) & ((1u << A.skip_bits) - 1));
            }
            uint32_t w = 0;
            if (EP == 1 && S.fast == 2) {   // the accumulator itself: the tables hold the bias and its unit
                const v4i fa = *(const v4i *)(tab + 64 * EPI_FA + 4 * q), fb = *(const v4i *)(tab + 64 * EPI_FB + 4 * q);
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    w |= (uint32_t)quant_f32((float)fin[IG * jj + q][e], __int_as_float(fa[e]), __int_as_float(fb[e]),
                                             (float)A.qmax) << (e * A.bits_out);
            } else if (S.fast) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    int u = v[jj][e];
                    if constexpr (EP == 2) {   // u fits in int32: sums modulo 2^32 are exact
                        const int scaled = rsm32(ss[e] ? u : kv[e], sc[e], sd[e]);
                        u = (int)((unsigned)scaled + (unsigned)(ss[e] ? kv[e] : u));
                    }
                    int y = requant32(u, mult[e], requant_rnd(shift[e]), shift[e] - 1);
                    y = y < 0 ? 0 : (y > A.qmax ? A.qmax : y);
                    w |= (uint32_t)y << (e * A.bits_out);
                }
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    long long u = v[jj][e];
                    if constexpr (EP == 2)
                        u = align_add(v[jj][e], kv[e], sc[e], sd[e], ss[e]);
                    w |= requant_clamp(u, mult[e], shift[e], A.qmax) << (e * A.bits_out);
                }
            }
            word[jj][q] = w;
        }
    }
    if constexpr (EP == 0)
        return;
    // 4 * IG codes: one store where a row of the tensor keeps them aligned
    // (cout a multiple of 4 * IG: the group is then all inside), else one
    // store of 1, 2 or 4 bytes per 4 codes
#pragma unroll
    for (int jj = 0; jj < JU; ++jj) {
        if (!ok[jj])
            continue;
        uint32_t (&w)[IG] = word[jj];
        const long long at = (px0 + 16 * jj) * A.cout + c0;
        if (A.bits_out == 4) {
            uint8_t *y = (uint8_t *)S.y + at / 2;
            if (IG == 4 && A.cout % 16 == 0) {
                *(uint2 *)y = make_uint2(w[0] | w[1 % IG] << 16, w[2 % IG] | w[3 % IG] << 16);
            } else if (IG == 2 && A.cout % 8 == 0) {
                *(uint32_t *)y = w[0] | w[1 % IG] << 16;
            } else {
#pragma unroll
                for (int q = 0; q < IG; ++q)
                    if (c0 + 4 * q < A.cout)
                        *(uint16_t *)(y + 2 * q) = (uint16_t)w[q];
            }
        } else if (A.bits_out == 2) {
            uint8_t *y = (uint8_t *)S.y + at / 4;
            if (IG == 4 && A.cout % 16 == 0) {
                *(uint32_t *)y = w[0] | w[1 % IG] << 8 | w[2 % IG] << 16 | w[3 % IG] << 24;
            } else if (IG == 2 && A.cout % 8 == 0) {
                *(uint16_t *)y = (uint16_t)(w[0] | w[1 % IG] << 8);
            } else {
#pragma unroll
                for (int q = 0; q < IG; ++q)
                    if (c0 + 4 * q < A.cout)
                        y[q] = (uint8_t)w[q];
            }
        } else {
            uint8_t *y = (uint8_t *)S.y + at;
            if (IG == 4 && A.cout % 16 == 0) {
                *(uint4 *)y = make_uint4(w[0], w[1 % IG], w[2 % IG], w[3 % IG]);
            } else {
#pragma unroll
                for (int q = 0; q < IG; ++q)
                    if (c0 + 4 * q < A.cout)
                        *(uint32_t *)(y + 4 * q) = w[q];
            }
        }
    }
}

template <int KIND, int MI, int NJ, int KW>
hipError_t launch_ep(const MfmaArgs &a, hipStream_t stream)
{
    const dim3 grid(8 * a.tiles_per_xcd), block(64 * KW);
    if (a.bits_out == 32)
        hipLaunchKernelGGL((qconv_gf_kernel<KIND, MI, NJ, KW, 0>), grid, block, 0, stream, a);
    else if (a.skip_bits == 0)
        hipLaunchKernelGGL((qconv_gf_kernel<KIND, MI, NJ, KW, 1>), grid, block, 0, stream, a);
    else
        hipLaunchKernelGGL((qconv_gf_kernel<KIND, MI, NJ, KW, 2>), grid, block, 0, stream, a);
    return hipGetLastError();
}

template <int KIND>
hipError_t launch_kind(const MfmaArgs &a, const GfPlan &p, hipStream_t stream)
{
    switch (p.mi * 100 + p.nj * 10 + p.kw) {
    case 441: return launch_ep<KIND, 4, 4, 1>(a, stream);
    case 442: return launch_ep<KIND, 4, 4, 2>(a, stream);
    case 444: return launch_ep<KIND, 4, 4, 4>(a, stream);
    case 421: return launch_ep<KIND, 4, 2, 1>(a, stream);
    case 422: return launch_ep<KIND, 4, 2, 2>(a, stream);
    case 424: return launch_ep<KIND, 4, 2, 4>(a, stream);
    case 144: return launch_ep<KIND, 1, 4, 4>(a, stream);
    case 224: return launch_ep<KIND, 2, 2, 4>(a, stream);
    }
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_qconv_gf(const MfmaArgs &a, const GfPlan &p, hipStream_t stream)
{
    const bool i8 = p.kind == GF_I8, f4 = p.kind == GF_F4;
    const int chunk = i8 ? 16 : 32, wb = p.kind == GF_F6 ? GF_F6_TILE : 1024;
    if (a.ksplit != 1 || a.part != 0 || a.kh > 7 || a.kw > 7 || a.cin % chunk != 0 ||
        a.ksteps != (a.kh * a.kw * (a.cin / chunk) + 3) / 4 || a.cout_pad % 64 != 0 || a.cout > a.cout_pad ||
        (a.bits_out != 32 && a.cout % 4 != 0) || (long long)a.ksteps * 4 * wb >= (1LL << 31))
        return hipErrorInvalidValue;
    // 32-bit buffer offsets and pixel numbers
    for (int i = 0; i < a.nseg; ++i)
        if ((long long)a.seg[i].n * a.seg[i].h * a.seg[i].w * (i8 ? a.cin : f4 ? a.cin / 4 : a.cin / 2) >= (1LL << 31) ||
            a.seg[i].P + 64 >= (1LL << 31))
            return hipErrorInvalidValue;
    switch (p.kind) {
    case GF_F6: return launch_kind<GF_F6>(a, p, stream);
    case GF_F4: return launch_kind<GF_F4>(a, p, stream);
    case GF_I8: return launch_kind<GF_I8>(a, p, stream);
    }
    return hipErrorInvalidValue;
}

}  // namespace aqd
