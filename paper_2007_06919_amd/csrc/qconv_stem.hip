// The 7x7 stride-2 input convolution (ResNet-50 stem) of the paper's fully
// quantized networks (Sec. 4: input and output layers at 8 bits): 8-bit codes
// of a 3-channel image, 8-bit two's-complement weights, on the int8 MFMA
// (v_mfma_i32_16x16x64_i8). GEMM view of Eq. 4 (Sec. 3.2.1): rows = output
// channels, columns = output pixels, K = the 7 x 7 x 3 window.
//
// With three input channels a K step cannot be a tap's channels, so the K axis is
// the whole window: 8 window rows (the last meets zero weights) of 8 taps (the last
// likewise) of 4 bytes (3 channels and a byte whose weight is zero), 256 = 4 K
// steps of two window rows. In LDS the image is held the same way, 4 bytes a
// pixel, re-centred as a - 128 like the other 8-bit path (the bias folded at
// create carries 128 * sum(w)): a window row then is 32 bytes from an 8-byte
// aligned address, whatever the pixel, and the MFMA's fragments are read straight
// from the image. Taps outside the image are code 0 (-128 after re-centring, as the
// correction assumes).
//
// Tile 64 channels x 8 rows of 32 output pixels: 21 rows of 69 image pixels, staged
// in pieces of 4 pixels (12 bytes: four dword loads, six shifts, one 16-byte LDS
// write), at most two a thread. Building every pixel's window in LDS instead, 49
// loads and 42 LDS writes a pixel on its own, is what bound the kernel before.
// Workgroups are persistent: each walks a contiguous range of tiles with its weights
// (16 KiB) and tables in LDS, the next tile's pieces in flight during
// this one's MFMAs and epilogue, two image buffers, one barrier a tile.
//
// 4 waves; wave w owns output rows 2w and 2w + 1 of the tile (4 column tiles of 16
// pixels) and all 64 channels (4 accumulator tiles). A row's K steps read the
// fragments of the row above one step later: 10 fragments serve 16 uses. Lane group
// g holds channels 16g .. 16g+15 of a pixel (rows permuted at create), one 8-byte
// store of 4-bit codes or four 16-byte stores of int32.
//
// Eight 800 x 1333 images: about 111 us with windows built in LDS, 58 here, 52 with the
// next tile found by counting instead of three divisions, no masks for tiles inside the
// image and the bias in the fp32 requantisation's b (93 MB, 1.8 TB/s); with the weights in
// registers instead of LDS the fp32 epilogue spilled, 94. What is left is instruction
// issue, the epilogue's five instructions a code above all: at the rates of an int8 MFMA
// loop and of a copy the matrix cores need about 20 us and the memory 17.

#include "epilogue.h"
#include "internal.h"
#include "mfma_common.h"

namespace aqd {
namespace {

typedef uint32_t dwords4 __attribute__((ext_vector_type(4), aligned(4)));

constexpr int ST_BCO = 64;                           // channels per tile
constexpr int ST_TW = STEM_TW, ST_TH = STEM_TH;      // output pixels of a tile: 32 x 8
constexpr int ST_CP = 18;                            // pieces of 4 image pixels per staged row
constexpr int ST_ROW = 16 * ST_CP;                   // LDS bytes per staged row
constexpr int ST_IR = 2 * ST_TH + 5;                 // staged rows (a last one is read against zero weights)
constexpr int ST_BUF = (ST_IR + 1) * ST_ROW;
constexpr int ST_NP = (ST_IR * ST_CP + 255) / 256;   // pieces per thread
static_assert(4 * ST_CP >= 2 * ST_TW + 6 && ST_TW == 32 && ST_TH == 8, "window of the last pixel");

// OUTK: 0 = 4-bit codes, 1 = int32 (v = acc + bias); FAST: 1 = every shift >= 2
// (32-bit requantisation), 2 = fp32 requantisation
template <int OUTK, int FAST>
__global__ void __launch_bounds__(256, OUTK == 0 && FAST == 1 ? 2 : 3) qconv_stem_kernel(MfmaArgs A)
{
    constexpr int MI = 4, QMAX = 15;
    __shared__ __attribute__((aligned(1024))) uint8_t lds[2 * ST_BUF];
    __shared__ __attribute__((aligned(1024))) uint8_t wts[4 * MI * 1024];   // [K step][row tile][lane][16]
    __shared__ __attribute__((aligned(16))) int32_t tab[3][ST_BCO];   // bias; multiplier and shift, or a and b

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, g = lane >> 4;

    // this workgroup's tiles: consecutive ones, an XCD's workgroups side by side
    const int chunk = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
    const int t0 = (int)((long long)A.total_tiles * chunk / gridDim.x);
    const int t1 = (int)((long long)A.total_tiles * (chunk + 1) / gridDim.x);
    if (t0 >= t1)
        return;

    struct Tile {
        int s, ct, n, oh, ow;
    };
    auto locate = [&](int tile) {
        Tile t{};
#pragma unroll
        for (int i = 1; i < AQD_MAX_SEGS; ++i)
            if (i < A.nseg && tile >= A.seg[i].tile_begin)
                t.s = i;
        const MfmaSeg &S = A.seg[t.s];
        // channel tiles outermost: the weights change rarely
        const unsigned tx = (unsigned)(S.wo + ST_TW - 1) / ST_TW, ty = (unsigned)(S.ho + ST_TH - 1) / ST_TH;
        const unsigned per = tx * ty * (unsigned)S.n, u = (unsigned)(tile - S.tile_begin);
        t.ct = (int)(u / per);
        const unsigned px = u - (unsigned)t.ct * per, row = px / tx;
        t.ow = (int)(px - row * tx) * ST_TW;
        t.n = (int)(row / ty);
        t.oh = (int)(row - (unsigned)t.n * ty) * ST_TH;
        return t;
    };

    // the tile after t (divisions are for the first one only)
    auto advance = [&](Tile t) {
        const MfmaSeg &S = A.seg[t.s];
        t.ow += ST_TW;
        if (t.ow >= S.wo) {
            t.ow = 0;
            t.oh += ST_TH;
            if (t.oh >= S.ho) {
                t.oh = 0;
                if (++t.n == S.n) {
                    t.n = 0;
                    if (++t.ct == A.co_tiles) {
                        t.ct = 0;
                        ++t.s;
                    }
                }
            }
        }
        return t;
    };

    // ---- a thread's pieces of a tile: pixels 4c .. 4c + 3 of staged row y. info:
    // the shift to the first pixel's byte (bits 0-1) and which pixels lie in the image
    // (bits 4-7). Byte offsets in 32 bits: the image has fewer than 2^31 bytes,
    // checked on the host.
    dwords4 raw[ST_NP];
    int info[ST_NP];
    bool inner = false;   // every staged pixel of the loaded tile lies in the image (and another row follows)
    auto load = [&](const Tile &t) {
        const MfmaSeg &S = A.seg[t.s];
        const int total = S.n * S.h * S.w * 3;       // image bytes (>= 3)
        const int ih0 = 2 * t.oh - 3, iw0 = 2 * t.ow - 3;
        inner = ih0 >= 0 && ih0 + ST_IR < S.h && iw0 >= 0 && iw0 + 4 * ST_CP <= S.w;
        if (inner) {
            const int base = ((t.n * S.h + ih0) * S.w + iw0) * 3;
#pragma unroll
            for (int k = 0; k < ST_NP; ++k) {
                const int p = tid + 256 * k;
                const int y = p / ST_CP, c = p - y * ST_CP;
                const int b = base + y * (3 * S.w) + 12 * c;
                info[k] = b & 3;
                if (y < ST_IR)
                    raw[k] = *(const dwords4 *)(S.x + (b & ~3));
            }
            return;
        }
#pragma unroll
        for (int k = 0; k < ST_NP; ++k) {
            const int p = tid + 256 * k;
            const int y = p / ST_CP, c = p - y * ST_CP;
            const int ih = ih0 + y, iw = iw0 + 4 * c;
            raw[k] = dwords4{0, 0, 0, 0};
            info[k] = 0;
            if (y >= ST_IR || (unsigned)ih >= (unsigned)S.h || iw >= S.w || iw < -3)
                continue;
            const int b = ((t.n * S.h + ih) * S.w + iw) * 3, a0 = b & ~3;
            const int right = min(S.w - iw, 4), left = max(-iw, 0);
            info[k] = (b & 3) | (((1 << right) - 1) & ~((1 << left) - 1)) << 4;
            if (a0 >= 0 && a0 <= total - 16) {
                raw[k] = *(const dwords4 *)(S.x + a0);
            } else {
                // at either end of the images: the bytes inside, one by one
                uint32_t v[4] = {0, 0, 0, 0};
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int at = a0 + e;
                    if (at >= 0 && at < total)
                        v[e / 4] |= (uint32_t)S.x[at] << (8 * (e % 4));
                }
                raw[k] = dwords4{v[0], v[1], v[2], v[3]};
            }
        }
    };
    auto write = [&](int buf) {
#pragma unroll
        for (int k = 0; k < ST_NP; ++k) {
            const int p = tid + 256 * k;
            if (p >= ST_IR * ST_CP)
                continue;
            const uint32_t u0 = __builtin_amdgcn_alignbyte(raw[k].y, raw[k].x, info[k] & 3);
            const uint32_t u1 = __builtin_amdgcn_alignbyte(raw[k].z, raw[k].y, info[k] & 3);
            const uint32_t u2 = __builtin_amdgcn_alignbyte(raw[k].w, raw[k].z, info[k] & 3);
            const uint32_t px[4] = {u0, __builtin_amdgcn_alignbyte(u1, u0, 3), __builtin_amdgcn_alignbyte(u2, u1, 2), u2 >> 8};
            v4i o;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int in = inner ? -1 : __builtin_amdgcn_sbfe(info[k], 4 + e, 1);
                o[e] = (int)((px[e] & (uint32_t)in) ^ 0x80808080u);
            }
            *(v4i *)(lds + buf * ST_BUF + 16 * p) = o;   // rows are ST_CP pieces
        }
    };

    // ---- weights and tables of a channel tile, as they are stored
    auto load_channels = [&](const Tile &t) {
        const MfmaSeg &S = A.seg[t.s];
        const uint8_t *w = (const uint8_t *)S.wt + (long long)t.ct * sizeof(wts);
#pragma unroll
        for (int k = 0; k < (int)sizeof(wts); k += 4096)
            *(v4i *)(wts + k + 16 * tid) = *(const v4i *)(w + k + 16 * tid);
        if (tid < 3 * ST_BCO) {
            const int f = tid / ST_BCO;
            const int field = f == 0 ? EPI_BIAS : f == 1 ? (FAST == 2 ? EPI_FA : EPI_MULT) : (FAST == 2 ? EPI_FB : EPI_SHIFT);
            tab[f][tid % ST_BCO] = S.epi[field * A.cout_pad + t.ct * ST_BCO + tid % ST_BCO];
        }
    };

    Tile cur = locate(t0);
    load(cur);
    load_channels(cur);
    write(0);
    __syncthreads();
    int buf = 0;
    for (int t = t0; t < t1; ++t) {
        const MfmaSeg &S = A.seg[cur.s];
        const bool more = t + 1 < t1;
        const Tile next = more ? advance(cur) : cur;
        if (more)
            load(next);

        // ---- MFMAs: row pair k of the wave's five serves K step k of its first
        // output row and K step k - 1 of its second; the sums start at the bias
        v4i acc[MI][4];   // column tile 2 (output row) + (half of the tile's width)
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            v4i bias = {0, 0, 0, 0};   // (fp32 requantisation: in b)
            if constexpr (FAST != 2)
                bias = *(const v4i *)&tab[0][16 * g + 4 * i];
#pragma unroll
            for (int j = 0; j < 4; ++j)
                acc[i][j] = bias;
        }
        const uint8_t *win = lds + buf * ST_BUF + (4 * wave + (g >> 1)) * ST_ROW + 8 * r + 16 * (g & 1);
        v4i fa[2][MI];   // weights of K steps k - 1 and k
#pragma unroll
        for (int k = 0; k < 5; ++k) {
#pragma unroll
            for (int i = 0; i < MI && k < 4; ++i)
                fa[k % 2][i] = *(const v4i *)(wts + (k * MI + i) * 1024 + 16 * lane);
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const uint2 lo = *(const uint2 *)(win + 2 * k * ST_ROW + 128 * c);
                const uint2 hi = *(const uint2 *)(win + 2 * k * ST_ROW + 128 * c + 8);
                const v4i b = {(int)lo.x, (int)lo.y, (int)hi.x, (int)hi.y};
#pragma unroll
                for (int i = 0; i < MI; ++i) {
                    if (k < 4)
                        acc[i][c] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fa[k % 2][i], b, acc[i][c], 0, 0, 0);
                    if (k > 0)
                        acc[i][2 + c] =
                            __builtin_amdgcn_mfma_i32_16x16x64_i8(fa[(k + 1) % 2][i], b, acc[i][2 + c], 0, 0, 0);
                }
            }
        }
        __builtin_amdgcn_sched_barrier(0);   // (no table read before: registers)

        // ---- epilogue: lane group g holds channels 16g + 4i + e of its pixels; per
        // channel group i the table entries are read once for all four
        uint32_t out[4][2] = {};
        if constexpr (OUTK == 0) {
#pragma unroll
            for (int i = 0; i < MI; ++i) {
                const v4i pa = *(const v4i *)&tab[1][16 * g + 4 * i], pb = *(const v4i *)&tab[2][16 * g + 4 * i];
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int v = acc[i][j][e];
                        int y;
                        if constexpr (FAST == 2) {
                            y = quant_f32((float)v, __int_as_float(pa[e]), __int_as_float(pb[e]), (float)QMAX);
                        } else if constexpr (FAST) {
                            y = requant32(v, pa[e], requant_rnd(pb[e]), pb[e] - 1);
                            y = y < 0 ? 0 : (y > QMAX ? QMAX : y);
                        } else {
                            y = (int)requant_clamp(v, pa[e], pb[e], QMAX);
                            asm volatile("" : "+v"(y));  // one 64-bit product alive at a time
                        }
                        const int bit = 4 * (4 * i + e);
                        out[j][bit >> 5] |= (uint32_t)y << (bit & 31);
                    }
            }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int oh = cur.oh + 2 * wave + (j >> 1), ow = cur.ow + 16 * (j & 1) + r;
            if (oh >= S.ho || ow >= S.wo)
                continue;
            const long long px = ((long long)cur.n * S.ho + oh) * S.wo + ow;
            const int c0 = cur.ct * ST_BCO + 16 * g;
            if constexpr (OUTK == 1) {
#pragma unroll
                for (int i = 0; i < MI; ++i)
                    *(v4i *)((int32_t *)S.y + px * A.cout + c0 + 4 * i) = acc[i][j];
            } else {
                *(uint2 *)((uint8_t *)S.y + (px * A.cout + c0) / 2) = make_uint2(out[j][0], out[j][1]);
            }
        }

        if (!more)
            break;
        write(buf ^ 1);    // (last read before the barrier of the tile before)
        if (next.s != cur.s || next.ct != cur.ct) {
            __syncthreads();   // every wave is done with the tables
            load_channels(next);
        }
        __syncthreads();
        cur = next;
        buf ^= 1;
    }
}

}  // namespace

hipError_t launch_qconv_stem(const MfmaArgs &a, hipStream_t stream)
{
    for (int i = 0; i < a.nseg; ++i)
        if ((long long)a.seg[i].n * a.seg[i].h * a.seg[i].w * 3 >= (1LL << 31))
            return hipErrorInvalidValue;   // byte offsets of the image in 32 bits
    if (a.cin != 3 || a.kh != 7 || a.kw != 7 || a.stride != 2 || a.pad != 3 || a.skip_bits != 0 ||
        (a.bits_out != 4 && a.bits_out != 32) || a.cout % ST_BCO != 0 || a.co_tiles * ST_BCO != a.cout ||
        a.ksplit != 1 || a.part != 0)
        return hipErrorInvalidValue;
    // three workgroups per CU, each with its share of the tiles
    dim3 grid(8 * (a.tiles_per_xcd < 96 ? a.tiles_per_xcd : 96)), block(256);
    int fast = 2;
    for (int i = 0; i < a.nseg; ++i)
        fast = a.seg[i].fast < fast ? a.seg[i].fast : fast;
    if (a.bits_out == 32)
        hipLaunchKernelGGL((qconv_stem_kernel<1, 1>), grid, block, 0, stream, a);
    else if (fast == 2)
        hipLaunchKernelGGL((qconv_stem_kernel<0, 2>), grid, block, 0, stream, a);
    else if (fast)
        hipLaunchKernelGGL((qconv_stem_kernel<0, 1>), grid, block, 0, stream, a);
    else
        hipLaunchKernelGGL((qconv_stem_kernel<0, 0>), grid, block, 0, stream, a);
    return hipGetLastError();
}

}  // namespace aqd
