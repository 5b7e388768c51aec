// Standalone integer skip connection (Sec. 3.2.3, Eq. 7) with nearest 2x
// upsample of the coarser operand (Sec. 3.2.4), and exact per-channel sums of
// an int32 tensor (the statistics a BN layer keeps, Sec. 3.2.2).

#include "epilogue.h"
#include "internal.h"

namespace aqd {
namespace {

__device__ __forceinline__ int load_value(const void *base, long long pix, int c, int ch, int bits)
{
    if (bits == 32)
        return ((const int32_t *)base)[pix * c + ch];
    return load_code((const uint8_t *)base + pix * (c * bits / 8), ch, bits);
}

// One thread per output byte: 8 / b_out channels of one pixel.
__global__ void __launch_bounds__(256) qadd_kernel(QaddArgs A)
{
    const int per = 8 / A.bits_out;
    const int groups = A.c / per;
    const long long P = (long long)A.n * A.h * A.w;
    const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= P * groups)
        return;
    const long long px = idx / groups;
    const int grp = (int)(idx - px * groups);
    long long bpix = px;
    if (A.up2) {
        const int hw = A.h * A.w;
        const int n = (int)(px / hw);
        const int rem = (int)(px - (long long)n * hw);
        const int y = rem / A.w, x = rem - y * A.w;
        bpix = ((long long)n * A.hb + (y >> 1)) * A.wb + (x >> 1);
    }
    const int qmax = A.qmax;
    uint32_t packed = 0;
    for (int e = 0; e < per; ++e) {
        const int ch = grp * per + e;
        const int a = load_value(A.a, px, A.c, ch, A.bits_a);
        const int b = load_value(A.b, bpix, A.c, ch, A.bits_b);
        const long long u = align_add(a, b, A.skip_c[ch], A.skip_d[ch], A.skip_side[ch]);
        packed |= requant_clamp(u, A.mult[ch], A.shift[ch], qmax) << (e * A.bits_out);
    }
    A.y[px * (A.c * A.bits_out / 8) + grp] = (uint8_t)packed;
}

// Workgroup: 256 consecutive channels x a strip of rows; int64 partial sums
// per thread, one atomic add per channel and workgroup (integer addition is
// associative, so the result is exact and order independent).
__global__ void __launch_bounds__(256) channel_sums_kernel(const int32_t *v, long long rows, int c,
                                                          long long rows_per_block, long long *sums)
{
    const int ch = blockIdx.x * 256 + threadIdx.x;
    if (ch >= c)
        return;
    const long long r0 = (long long)blockIdx.y * rows_per_block;
    long long r1 = r0 + rows_per_block;
    if (r1 > rows)
        r1 = rows;
    long long s1 = 0, s2 = 0;
    for (long long r = r0; r < r1; ++r) {
        const long long x = v[r * c + ch];
        s1 += x;
        s2 += x * x;
    }
    atomicAdd((unsigned long long *)&sums[ch], (unsigned long long)s1);
    atomicAdd((unsigned long long *)&sums[c + ch], (unsigned long long)s2);
}

// The same with 16-byte loads, for channel counts that are a multiple of 4 and a
// 16-byte aligned tensor. One thread per channel walks its rows one load after
// another, with too few rows in flight to reach the memory's rate (16700 x 256:
// 71 us, 0.24 TB/s). Here a thread takes 4 channels of every 16th row of the strip,
// four rows in flight, and the sixteen row groups are added in LDS. The strips'
// atomics then set the pace (512 strips of 4 row groups: 47 us), so there are few
// strips, each on a workgroup of 16 waves.
constexpr int CS_TY = 16;
__global__ void __launch_bounds__(64 * CS_TY) channel_sums4_kernel(const int32_t *v, long long rows, int c,
                                                                  long long rows_per_block, long long *sums)
{
    __shared__ long long part[CS_TY][64][2];
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
    const int ch = (blockIdx.x * 64 + tx) * 4;
    const long long r0 = (long long)blockIdx.y * rows_per_block;
    const long long r1 = r0 + rows_per_block < rows ? r0 + rows_per_block : rows;
    long long s[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    auto add = [&](const int4 x) {
        const int e[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            s[k] += e[k];
            s[4 + k] += (long long)e[k] * e[k];
        }
    };
    if (ch < c) {
        const int32_t *p = v + ch;
        long long r = r0 + ty;
        for (; r + 3 * CS_TY < r1; r += 4 * CS_TY) {
            int4 x[4];
#pragma unroll
            for (int k = 0; k < 4; ++k)
                x[k] = *(const int4 *)(p + (r + k * CS_TY) * c);
#pragma unroll
            for (int k = 0; k < 4; ++k)
                add(x[k]);
        }
        for (; r < r1; r += CS_TY)
            add(*(const int4 *)(p + r * c));
    }
    // channel k of each four: row group 0 adds up the sums, row group 1 the squares
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        __syncthreads();
        part[ty][tx][0] = s[k];
        part[ty][tx][1] = s[4 + k];
        __syncthreads();
        if (ty < 2 && ch < c) {
            long long t = 0;
#pragma unroll
            for (int y = 0; y < CS_TY; ++y)
                t += part[y][tx][ty];
            atomicAdd((unsigned long long *)&sums[ty * c + ch + k], (unsigned long long)t);
        }
    }
}

}  // namespace

hipError_t launch_qadd(const QaddArgs &a, hipStream_t stream)
{
    const long long total = (long long)a.n * a.h * a.w * (a.c / (8 / a.bits_out));
    if (total == 0)
        return hipSuccess;
    const long long blocks = (total + 255) / 256;
    if (blocks > 0x7fffffffLL)
        return hipErrorInvalidValue;
    hipLaunchKernelGGL(qadd_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, a);
    return hipGetLastError();
}

hipError_t launch_channel_sums(const int32_t *v, long long rows, int c, long long *sums,
                               hipStream_t stream)
{
    if (rows == 0)
        return hipSuccess;
    if (c % 4 == 0 && ((uintptr_t)v & 15) == 0) {
        const int gx = (c / 4 + 63) / 64;
        // about 96 workgroups: more add atomics to the same few sums (each takes its turn),
        // fewer leave the rows' loads too few in flight. us, rows from HBM, at 24 / 48 / 96 /
        // 192 / 384 workgroups: 4200 x 256 10.8 / 10.5 / 11.5 / 11.5 / 11.5; 16700 x 256
        // 22.4 / 16.7 / 18.5 / 25.9 / 31.3; 67000 x 256 69.7 / 43.2 / 35.0 / 42.4 / 53.0;
        // 267200 x 256 262 / 152 / 102 / 103 / 99; 267200 x 64 153 / 86 / 53 / 45 / 55;
        // 33600 x 1024 125 / 73 / 49 / 47 / 47
        const long long strips = 96 / gx > 8 ? 96 / gx : 8;
        long long per = (rows + strips - 1) / strips;
        per = per < 64 ? 64 : per;
        hipLaunchKernelGGL(channel_sums4_kernel, dim3(gx, (unsigned)((rows + per - 1) / per)), dim3(64 * CS_TY), 0,
                           stream, v, rows, c, per, sums);
        return hipGetLastError();
    }
    // at most 4096 row strips (grid.y limit is 65535)
    long long rows_per_block = (rows + 4095) / 4096;
    if (rows_per_block < 256)
        rows_per_block = 256;
    const long long ystrips = (rows + rows_per_block - 1) / rows_per_block;
    dim3 grid((c + 255) / 256, (unsigned)ystrips);
    hipLaunchKernelGGL(channel_sums_kernel, grid, dim3(256), 0, stream, v, rows, c, rows_per_block,
                       sums);
    return hipGetLastError();
}

}  // namespace aqd
