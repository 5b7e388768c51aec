// Implicit-GEMM integer convolution of 8-bit codes (the input and output layers of
// the paper's fully quantized networks, Sec. 4) on the int8 MFMA
// (v_mfma_i32_16x16x64_i8, K step = 64 input channels), for cin a multiple of 128 and
// int32 outputs (the prediction convolutions). GEMM view of Eq. 4 (Sec. 3.2.1): rows =
// output channels, columns = output pixels, K = taps x input channels.
//
// Exactness. An 8-bit code a in [0, 255] does not fit int8; the staging copy stores
// a - 128 (the byte a XOR 0x80, read as signed), padding taps included (code 0 ->
// -128), and the bias folded at create carries 128 * sum(w) of the channel, so
// v = acc + bias is the exact sum of Eq. 6.
//
// Workgroup tile 256 channels x 128 pixels, 4 waves; wave w owns channel rows
// 64w .. 64w+63 (4 accumulator tiles of 16) for all 128 pixels (8 column
// tiles), as in the register-fed int8 kernel:
//  * weights (tiled at create, 64 bytes per row and K step) go from global memory
//    straight into registers, three K steps ahead of their MFMAs;
//  * activation codes go through LDS in stages of 128 bytes per pixel (one tap's 128
//    channels; two K steps), 16 bytes per copy lane. A pixel's 128 bytes are 16-byte
//    columns XOR-swizzled with the pixel index, so that the copies' writes and the
//    fragment reads (16 bytes per lane) are free of bank conflicts. A stage is loaded
//    one stage ahead of its use and written during the stage before it (two-buffer
//    ring, one barrier per stage).
//  * A part of a split K range (whole stages) writes int32 partial sums, the
//    first part with the bias, for the split-K combining epilogue.

#include "internal.h"
#include "mfma_common.h"

namespace aqd {
namespace {

constexpr int B8_BCO = 256;                   // channels per workgroup tile
constexpr int B8_BPX = 128;                   // pixels per workgroup tile
constexpr int B8_ROW = 128;                   // LDS bytes of one stage per pixel
constexpr int B8_STAGE = B8_BPX * B8_ROW;     // 16 KiB
constexpr int B8_LDS = 4 * B8_STAGE;          // a ring of two stages; the outputs use all 64 KiB
constexpr int B8_KROW = 64;                   // weight bytes per row and K step

// v = acc + bias, or a split part's sums
__global__ void __launch_bounds__(256, 2) qconv_b8_kernel(MfmaArgs A)
{
    constexpr int MI = 4, NJ = 8;
    constexpr int SPS = 2;                      // 64-channel steps per stage
    constexpr int SCH = 128;                    // input channels per stage
    __shared__ __attribute__((aligned(1024))) uint8_t lds[B8_LDS];

    const int bid = blockIdx.x;
    const int logical = (bid & 7) * A.tiles_per_xcd + (bid >> 3);
    if (logical >= A.total_tiles)
        return;
    // work unit -> output tile and part of its K range (consecutive units)
    const int tile = logical / A.ksplit;
    const int kpart = logical - tile * A.ksplit;
    int s = 0;
#pragma unroll
    for (int i = 1; i < AQD_MAX_SEGS; ++i)
        if (i < A.nseg && tile >= A.seg[i].tile_begin)
            s = i;
    const MfmaSeg &S = A.seg[s];
    const int t_in_seg = tile - S.tile_begin;
    const int co_tile = t_in_seg % A.co_tiles;
    const int px_tile = t_in_seg / A.co_tiles;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, g = lane >> 4;

    // K range of this part in stages (one tap's SCH channels; A.ksteps and
    // A.kchunk count 64-channel steps, multiples of SPS on this path); the
    // kernel's K steps are two per stage
    const int row_bytes = A.cin;
    const int spt = A.cin / SCH;                           // stages per tap
    const int st0 = kpart * (A.kchunk / SPS);
    const int NST = min(A.kchunk, A.ksteps - kpart * A.kchunk) / SPS;  // >= 1 (host)
    const int KSK = 2 * (A.ksteps / SPS);                  // kernel K steps of the whole range
    const int hw = S.ho * S.wo;

    // ---- activation copies: piece m of a stage = pixels 32m .. 32m+31, lane
    // tid copying stage bytes 16c .. 16c+15 of pixel 32m + tid / 8, c = tid % 8
    const int c8 = tid & 7;
    // per piece: the byte offset of its pixel's window origin (negative at the
    // top and left borders) and which window rows (bit t) and columns (bit
    // 16 + t) lie inside the image (none for pixels past the end); the input
    // holds n * h * w * row_bytes < 2^31 bytes (checked on the host)
    int xbase[4];
    uint32_t xvalid[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) {
        const unsigned p = (unsigned)(px_tile * B8_BPX + 32 * m + (tid >> 3));
        const bool ok = p < (unsigned)S.P;
        const unsigned pn = ok ? p / (unsigned)hw : 0u;
        const unsigned prem = ok ? p - pn * (unsigned)hw : 0u;
        const int oh = (int)(prem / (unsigned)S.wo), ow = (int)prem - oh * S.wo;
        const int ih0 = oh * A.stride - A.pad, iw0 = ow * A.stride - A.pad;
        uint32_t v = 0;
        for (int t = 0; t < A.kh; ++t)
            v |= ((unsigned)(ih0 + t) < (unsigned)S.h ? 1u : 0u) << t;
        for (int t = 0; t < A.kw; ++t)
            v |= ((unsigned)(iw0 + t) < (unsigned)S.w ? 1u : 0u) << (16 + t);
        xvalid[m] = ok ? v : 0u;
        xbase[m] = (((int)pn * S.h + ih0) * S.w + iw0) * row_bytes + 16 * c8;
    }
    const buf_rsrc xr = make_rsrc(S.x, S.n * S.h * S.w * row_bytes);
    // LDS: 16-byte column c of pixel p at 128 p + 16 (c ^ (p & 7))
    const int wp = tid >> 3;
    const uint32_t wofs = B8_ROW * wp + 16 * (c8 ^ (wp & 7));
    // fragment of K step q of a stage: pixel 16j + r, column 4q + g
    auto ro = [&](int q) -> uint32_t { return B8_ROW * r + 16 * ((4 * q + g) ^ (r & 7)); };

    // copy state of the stage being loaded (uniform): tap (tr, tq), SCH-channel
    // chunk th; its byte offset from a window origin and the window bits it needs
    int th = st0 % spt, tr, tq;
    {
        const int tap = st0 / spt;
        tr = tap / A.kw;
        tq = tap - tr * A.kw;
    }
    int x_off = 0;
    uint32_t x_need = 0;
    auto set_copy = [&]() {
        x_off = (tr * S.w + tq) * row_bytes + SCH * th;
        x_need = (1u << tr) | (1u << (16 + tq));
    };
    set_copy();
    auto advance = [&]() {
        if (++th == spt) {
            th = 0;
            if (++tq == A.kw) {
                tq = 0;
                ++tr;
            }
        }
        set_copy();
    };
    // buffer loads: taps in the padding, pixels past the end and stages past
    // the last read past the end of the input and get zeros (code 0)
    auto load_piece = [&](int m) -> v4i {
        return load_b128(xr, (xvalid[m] & x_need) == x_need ? xbase[m] + x_off : (int)0x80000000, 0);
    };
    // code a -> a - 128
    auto write_piece = [&](int buf, int m, const v4i v) {
        const int flip = (int)0x80808080u;
        *(v4i *)(lds + buf * B8_STAGE + m * (32 * B8_ROW) + wofs) = v ^ v4i{flip, flip, flip, flip};
    };

    // ---- weights: this wave's rows of K step k, accumulator tile i at
    // k * 16 KiB + i * 1 KiB from the channel tile's first step (lane: row r,
    // 16-byte column g); the look-ahead reads up to three steps past the
    // part's last (inside the tile range, or past the buffer's size: zeros),
    // never used
    const buf_rsrc wr = make_rsrc(S.wt + (long long)co_tile * KSK * B8_BCO * B8_KROW, KSK * B8_BCO * B8_KROW);
    const int w_lane = (64 * wave + r) * B8_KROW + 16 * g;
    const int k0 = 2 * st0;
    auto load_a = [&](int k, v4i *dst) {
#pragma unroll
        for (int i = 0; i < MI; ++i)
            dst[i] = load_b128(wr, w_lane + i * 1024, (k0 + k) * (B8_BCO * B8_KROW));
    };

    // lane group g of wave w holds channels 128 (w >> 1) + 32 g + 16 (w & 1) + 4 i + e
    const int co_loc = 128 * (wave >> 1) + 32 * g + 16 * (wave & 1);
    const int co_glob = co_tile * B8_BCO + co_loc;
    v4i acc[MI][NJ];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
            acc[i][j] = v4i{0, 0, 0, 0};

    // ---- prologue: stage 0 in LDS, stage 1 in registers, weights of steps 0-2
    v4i rb[4];
#pragma unroll
    for (int m = 0; m < 4; ++m)
        write_piece(0, m, load_piece(m));
    advance();
#pragma unroll
    for (int m = 0; m < 4; ++m)
        rb[m] = load_piece(m);
    advance();  // copy state: stage 2
    v4i fa[4][MI];
    load_a(0, fa[0]);
    load_a(1, fa[1]);
    load_a(2, fa[2]);
    v4i fb[NJ];
    int kstep = 0;         // K step of this part being multiplied
    constexpr int RA = 2;  // fragments are read RA column tiles ahead of their MFMAs
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
    for (int j = 0; j < RA; ++j)
        fb[j] = *(const v4i *)(lds + 2048 * j + ro(0));

    // ---- main loop, one stage (two K steps) per call: stage t lives in buffer
    // t % 2 (the parity P, a compile-time constant, so that the weight sets
    // (K step % 4) are registers). During stage t the pieces of stage t + 1
    // (loaded during stage t - 1) are written into buffer (t + 1) % 2, two per
    // K step, each right before the load of the same piece of stage t + 2
    // reuses its registers. The barrier in the last K step, before the first
    // read of stage t + 1, makes that stage visible; every read of stage t - 1
    // (the buffer's previous contents) came before the barrier of stage t - 1.
    auto stage = [&](auto pc) {
        constexpr int P = decltype(pc)::value;
        static_for<2>([&](auto qc) {
            constexpr int q = decltype(qc)::value;
            constexpr int kq = 2 * P + q;  // K step % 4
            write_piece(P ^ 1, 2 * q, rb[2 * q]);
            write_piece(P ^ 1, 2 * q + 1, rb[2 * q + 1]);
            rb[2 * q] = load_piece(2 * q);
            rb[2 * q + 1] = load_piece(2 * q + 1);
            load_a(kstep + 3, fa[(kq + 3) & 3]);
            const uint32_t r_this = ro(q) + P * B8_STAGE;
            const uint32_t r_next = q == 0 ? ro(1) + P * B8_STAGE : ro(0) + (P ^ 1) * B8_STAGE;
            static_for<NJ>([&](auto jc) {
                constexpr int j = decltype(jc)::value;
                if constexpr (q == 1 && j == NJ - RA)
                    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
                for (int i = 0; i < MI; ++i)
                    acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fa[kq][i], fb[j], acc[i][j], 0, 0, 0);
                if constexpr (j + RA < NJ)
                    fb[j + RA] = *(const v4i *)(lds + 2048 * (j + RA) + r_this);
                else
                    fb[j + RA - NJ] = *(const v4i *)(lds + 2048 * (j + RA - NJ) + r_next);
            });
            ++kstep;
            if constexpr (q == 1)
                advance();
        });
    };
    // pairs of stages (even, odd parity); the odd stage of the last pair may
    // be past the end
    for (int t = 0; t < NST; t += 2) {
        stage(std::integral_constant<int, 0>{});
        if (t + 1 < NST)
            stage(std::integral_constant<int, 1>{});
    }

    // int32 outputs (or part sums at y + kpart * P * cout), in two passes
    // of 64 pixels through LDS rows of 256 int32 (16-byte chunk c of pixel
    // p at c ^ (p & 7)); every thread then stores 16-byte chunks of whole rows
    int32_t *ybase = (int32_t *)S.y + (long long)kpart * S.P * A.cout;
    // the tile's valid 16-byte chunks (a partial last channel tile)
    const int valid_chunks = min(A.cout - co_tile * B8_BCO, B8_BCO) / 4;
    const bool with_bias = !(A.part && kpart > 0);
    v4i bias[MI];
#pragma unroll
    for (int i = 0; i < MI; ++i)
        bias[i] = with_bias ? *(const v4i *)(S.epi + EPI_BIAS * A.cout_pad + co_glob + 4 * i) : v4i{0, 0, 0, 0};
    static_for<2>([&](auto pc) {
        constexpr int pass = decltype(pc)::value;
        __syncthreads();  // the ring, or the last pass's rows, are no longer read
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
            const int p = 16 * jj + r;
#pragma unroll
            for (int i = 0; i < MI; ++i) {
                const int c = co_loc / 4 + i;
                *(v4i *)(lds + p * 1024 + 16 * (c ^ (p & 7))) = acc[i][4 * pass + jj] + bias[i];
            }
        }
        __syncthreads();
#pragma unroll
        for (int it = 0; it < 16; ++it) {
            const int idx = it * 256 + tid;
            const int p = idx >> 6, c = idx & 63;
            const long long px = (long long)px_tile * B8_BPX + 64 * pass + p;
            if (px < S.P && c < valid_chunks)
                *(v4i *)(ybase + px * A.cout + co_tile * B8_BCO + 4 * c) =
                    *(const v4i *)(lds + p * 1024 + 16 * (c ^ (p & 7)));
        }
    });
}

}  // namespace

hipError_t launch_qconv_b8(const MfmaArgs &a, hipStream_t stream)
{
    dim3 grid(8 * a.tiles_per_xcd), block(256);
    // int32 outputs (or split parts); a partial last channel tile
    if ((a.part == 0 && a.ksplit != 1) || a.kh > 16 || a.kw > 16 || a.bits_out != 32 || a.skip_bits != 0 ||
        a.cin % 128 != 0 || a.co_tiles * B8_BCO < a.cout || a.cout % 4 != 0 || a.ksteps % 2 != 0 ||
        a.kchunk % 2 != 0 || a.kchunk < 2 || (long long)a.co_tiles * a.ksteps * B8_BCO * B8_KROW >= (1LL << 31))
        return hipErrorInvalidValue;
    // 32-bit buffer offsets and sizes: inputs and weights below 2^31 bytes
    for (int i = 0; i < a.nseg; ++i)
        if ((long long)a.seg[i].n * a.seg[i].h * a.seg[i].w * a.cin >= (1LL << 31))
            return hipErrorInvalidValue;
    hipLaunchKernelGGL(qconv_b8_kernel, grid, block, 0, stream, a);
    return hipGetLastError();
}

}  // namespace aqd
