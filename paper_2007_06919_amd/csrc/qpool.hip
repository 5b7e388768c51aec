// Max-pooling of b-bit code tensors (Sec. 3.2.4: pooling leaves the scale
// factor of its input unchanged, so the codes are pooled as they are, with no
// arithmetic beyond comparisons). Window positions outside the input are
// skipped (codes are >= 0, so this equals pooling over a zero-padded input
// whenever the window holds at least one input position, which the host
// checks).

#include "internal.h"

namespace aqd {
namespace {

// One thread per output byte: 8 / b channels of one output pixel (rows whose
// byte count is not a multiple of 16).
__global__ void __launch_bounds__(256) maxpool_kernel(PoolArgs A)
{
    const int per = 8 / A.bits;
    const int groups = A.c / per;
    const long long P = (long long)A.n * A.ho * A.wo;
    const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= P * groups)
        return;
    const long long px = idx / groups;
    const int grp = (int)(idx - px * groups);
    const int hw = A.ho * A.wo;
    const int n = (int)(px / hw);
    const int rem = (int)(px - (long long)n * hw);
    const int i = rem / A.wo, j = rem - i * A.wo;
    const int row_bytes = A.c * A.bits / 8;
    const int mask = (1 << A.bits) - 1;
    int best[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    for (int dy = 0; dy < A.k; ++dy) {
        const int ih = i * A.stride - A.pad + dy;
        if ((unsigned)ih >= (unsigned)A.h)
            continue;
        for (int dx = 0; dx < A.k; ++dx) {
            const int iw = j * A.stride - A.pad + dx;
            if ((unsigned)iw >= (unsigned)A.w)
                continue;
            const int v = A.x[(((long long)n * A.h + ih) * A.w + iw) * row_bytes + grp];
            for (int e = 0; e < per; ++e) {
                const int code = (v >> (e * A.bits)) & mask;
                best[e] = code > best[e] ? code : best[e];
            }
        }
    }
    uint32_t packed = 0;
    for (int e = 0; e < per; ++e)
        packed |= (uint32_t)best[e] << (e * A.bits);
    A.y[px * row_bytes + grp] = (uint8_t)packed;
}

// Running lane-wise maxima of packed b-bit codes: 16 / b accumulators per word,
// one per code of a 16-bit half, each the packed 16-bit maximum of that code in
// place (an unsigned comparison of values that differ in that code alone; the top
// code decides its comparison by itself, so it needs no mask until the end).
// 4-bit codes: 7 instructions a word and window position.
typedef unsigned short half2u __attribute__((ext_vector_type(2)));
template <int B>
struct PackedMax {
    static constexpr int N = 16 / B;
    static constexpr uint32_t M = (1u << B) - 1;
    half2u acc[N] = {};   // codes are >= 0, and the window holds an input position
    __device__ __forceinline__ static uint32_t mask(int i) { return (M | M << 16) << (B * i); }
    __device__ __forceinline__ void add(uint32_t v)
    {
#pragma unroll
        for (int i = 0; i < N; ++i)
            acc[i] = __builtin_elementwise_max(acc[i], __builtin_bit_cast(half2u, i < N - 1 ? v & mask(i) : v));
    }
    __device__ __forceinline__ uint32_t get() const
    {
        uint32_t out = 0;
#pragma unroll
        for (int i = 0; i < N; ++i)
            out |= __builtin_bit_cast(uint32_t, acc[i]) & mask(i);
        return out;
    }
};

// 16 bytes of one output pixel per thread (rows of a multiple of 16 bytes): one
// 16-byte load per window position and lane-wise maxima. K: the window, 0 = at run
// time; a known window's loads are all in flight at once. idx_t: unsigned while the
// items fit (a 64-bit division costs more than the maxima).
// 3 x 3 stride 2 over [8][400][667][64] 4-bit codes: 27.2 us with one load at a time,
// borrow-and-select maxima and 64-bit divisions, 19.0 here (85 MB, 4.5 TB/s; a copy
// reaches 5.4); one image 7.6 -> 5.4.
template <int B, int K, typename idx_t>
__global__ void __launch_bounds__(256) maxpool16_kernel(PoolArgs A)
{
    const idx_t chunks = A.c * B / 128;
    const idx_t items = (idx_t)A.n * A.ho * A.wo * chunks;
    const idx_t idx = (idx_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= items)
        return;
    const idx_t px = idx / chunks;
    const int ch = (int)(idx - px * chunks);
    const idx_t row = px / (idx_t)A.wo;
    const int j = (int)(px - row * (idx_t)A.wo);
    const int n = (int)(row / (idx_t)A.ho);
    const int i = (int)(row - (idx_t)n * (idx_t)A.ho);
    const int row_bytes = A.c * B / 8;
    const int ih0 = i * A.stride - A.pad, iw0 = j * A.stride - A.pad;
    const uint8_t *x = A.x + (((long long)n * A.h + ih0) * A.w + iw0) * row_bytes + 16 * ch;
    PackedMax<B> best[4];
    auto add = [&](const uint4 v) {
        best[0].add(v.x);
        best[1].add(v.y);
        best[2].add(v.z);
        best[3].add(v.w);
    };
    if constexpr (K > 0) {
        uint4 v[K][K];
#pragma unroll
        for (int dy = 0; dy < K; ++dy)
#pragma unroll
            for (int dx = 0; dx < K; ++dx) {
                v[dy][dx] = make_uint4(0, 0, 0, 0);
                if ((unsigned)(ih0 + dy) < (unsigned)A.h && (unsigned)(iw0 + dx) < (unsigned)A.w)
                    v[dy][dx] = *(const uint4 *)(x + ((long long)dy * A.w + dx) * row_bytes);
            }
#pragma unroll
        for (int dy = 0; dy < K; ++dy)
#pragma unroll
            for (int dx = 0; dx < K; ++dx)
                add(v[dy][dx]);
    } else {
        for (int dy = 0; dy < A.k; ++dy)
            for (int dx = 0; dx < A.k; ++dx)
                if ((unsigned)(ih0 + dy) < (unsigned)A.h && (unsigned)(iw0 + dx) < (unsigned)A.w)
                    add(*(const uint4 *)(x + ((long long)dy * A.w + dx) * row_bytes));
    }
    *(uint4 *)(A.y + (long long)px * row_bytes + 16 * ch) =
        make_uint4(best[0].get(), best[1].get(), best[2].get(), best[3].get());
}

template <int B>
void launch16(const PoolArgs &a, long long items, hipStream_t stream)
{
    const dim3 grid((unsigned)((items + 255) / 256)), block(256);
    if (items + 256 >= (1LL << 31))
        hipLaunchKernelGGL((maxpool16_kernel<B, 0, long long>), grid, block, 0, stream, a);
    else if (a.k == 3)
        hipLaunchKernelGGL((maxpool16_kernel<B, 3, unsigned>), grid, block, 0, stream, a);
    else
        hipLaunchKernelGGL((maxpool16_kernel<B, 0, unsigned>), grid, block, 0, stream, a);
}

}  // namespace

hipError_t launch_maxpool(const PoolArgs &a, hipStream_t stream)
{
    const int row_bytes = a.c * a.bits / 8;
    if (row_bytes % 16 == 0 && ((uintptr_t)a.x & 15) == 0 && ((uintptr_t)a.y & 15) == 0) {
        const long long items = (long long)a.n * a.ho * a.wo * (row_bytes / 16);
        if (items <= 0)
            return hipSuccess;
        if (a.bits == 2)
            launch16<2>(a, items, stream);
        else if (a.bits == 4)
            launch16<4>(a, items, stream);
        else
            launch16<8>(a, items, stream);
        return hipGetLastError();
    }
    const long long items = (long long)a.n * a.ho * a.wo * (a.c * a.bits / 8);
    if (items <= 0)
        return hipSuccess;
    hipLaunchKernelGGL(maxpool_kernel, dim3((unsigned)((items + 255) / 256)), dim3(256), 0, stream, a);
    return hipGetLastError();
}

}  // namespace aqd
