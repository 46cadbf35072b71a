// Fixed-order reductions that follow the GEMM kernels:
//  * rowsum_combine: adds the per-tile-column row-sum partials in tile order, in 64 bits;
//  * splitk_reduce: second pass of the split-K path -- adds the K-slice partial
//    products in slice order, then bias, activation, store and row sum.
// No atomics: equal inputs give bit-equal outputs.  Both read each
// summand once: bound by memory bandwidth when the output is large, by the latency of the loads when it is not.
#include <hip/hip_runtime.h>

#include "pgk_device.h"
#include "pgk_kernels.h"

namespace pgk {

// load(0) + load(1) + ... + load(n - 1), added in that order, up to eight loads in flight.  These passes
// are bound by the latency of their loads, and a loop of load and add pays it once per summand.  Whole call
// in a graph, before and after: 256 x 256 x 256 float32 7.5 and 6.6 us, 1 x 4096 x 4096 bf16 14.1 and
// 13.3, 32 x 8192 x 8192 bf16 with row sums 34.1 and 29.3 (8 x 11008 x 4096 bf16 the same within the noise).  The
// batches are of fixed sizes: one of eight guarded by s < n leaves a branch around each load, and two to
// four slices were slower for it (768 x 768 x 3072 bf16 21.0 and 23.1).
template <int BATCH, typename V, typename F>
__device__ __forceinline__ void ordered_batch(V& sum, int& s, F&& load)
{
    V v[BATCH];
#pragma unroll
    for (int q = 0; q < BATCH; ++q) v[q] = load(s + q);
#pragma unroll
    for (int q = 0; q < BATCH; ++q) sum += v[q];
    s += BATCH;
}
template <typename V, int FIRST = 8, typename F>
__device__ __forceinline__ V ordered_sum(int n, F&& load)
{
    V sum = load(0);
    int s = 1;
    if constexpr (FIRST > 8)
        while (n - s >= FIRST) ordered_batch<FIRST>(sum, s, load);
    while (n - s >= 8) ordered_batch<8>(sum, s, load);
    if (n - s >= 4) ordered_batch<4>(sum, s, load);
    if (n - s >= 2) ordered_batch<2>(sum, s, load);
    if (n - s >= 1) ordered_batch<1>(sum, s, load);
    return sum;
}

// In 64 bits: the partials are added one after another for each row, so their number, which goes by the tile's width,
// would otherwise show in the error (256 x 44864 x 3079, bf16 with odd rows: 176 columns of 256 2.1e-7, 351 of 128 2.8e-7; in 64 bits
// 2.8e-8).  Slower than 32-bit additions where few rows have hundreds of tile columns, which sixteen loads in flight more than make
// up for (whole calls, 32 bits / 64 bits / with sixteen loads: 100 x 30000 x 512 fp32 42.5, 43.2, 39.7 us, 300 x 40000 x 256 bf16 35.0, 35.2,
// 32.8, 64 x 50000 x 200 fp32 50.0, 50.8, 39.1); added in pairs 43.0, 35.9 and 51.4.
__global__ __launch_bounds__(256) void rowsum_combine_kernel(const float* __restrict__ part,
                                                             float* __restrict__ rowsum,
                                                             int M, int batch, int tiles_n)
{
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    const size_t total = (size_t)M * batch;
    if (i >= total) return;
    const size_t b = i / M, m = i - b * M;
    const float* src = part + b * (size_t)tiles_n * M + m;
    rowsum[i] = (float)ordered_sum<double, 16>(tiles_n, [&](int t) { return (double)src[(size_t)t * M]; });
}

hipError_t launch_rowsum_combine(const float* part, float* rowsum, int M, int batch, int tiles_n,
                                 hipStream_t s)
{
    const size_t total = (size_t)M * batch;
    const size_t blocks = (total + 255) / 256;
    if (blocks == 0 || blocks > 0x7fffffffULL) return hipErrorInvalidValue;
    hipLaunchKernelGGL(rowsum_combine_kernel, dim3((unsigned int)blocks), dim3(256), 0, s, part, rowsum, M,
                       batch, tiles_n);
    return hipGetLastError();
}

// One wave per output row and column segment (blockIdx.y; segments of seg_cols columns, so
// that skinny outputs still give enough waves).  VEC = 4 when N % 4 == 0 and the buffers are
// 16-byte aligned (each lane handles 4 consecutive columns per trip), else 1.  With several
// segments the row sums are per-segment partials rs_part[b][segment][m], to be added in
// segment order by rowsum_combine_kernel.
template <int VEC, bool OUT_BF16>
__global__ __launch_bounds__(256) void splitk_reduce_kernel(const float* __restrict__ ws,
                                                            const float* __restrict__ bias,
                                                            void* __restrict__ C, float* __restrict__ rowsum,
                                                            float* __restrict__ rs_part, int seg_cols,
                                                            int M, int N, int batch, int splits, int act)
{
    const int lane = threadIdx.x & 63;
    const size_t row = (size_t)blockIdx.x * 4 + (threadIdx.x >> 6);   // b * M + m
    if (row >= (size_t)M * batch) return;
    const int seg = blockIdx.y, nseg = gridDim.y;
    const int n_begin = seg * seg_cols;
    const int n_end = n_begin + seg_cols < N ? n_begin + seg_cols : N;
    const size_t b = row / M, m = row - b * M;
    const size_t slice = (size_t)M * N;
    const float* src = ws + b * (size_t)splits * slice + m * (size_t)N;
    const size_t out = row * (size_t)N;

    float rs = 0.0f;
    for (int n = n_begin + lane * VEC; n < n_end; n += 64 * VEC) {
        float x[VEC], add[VEC];
#pragma unroll
        for (int e = 0; e < VEC; ++e) add[e] = bias ? bias[n + e] : 0.0f;
        if constexpr (VEC == 4) {
            const f32x4 v = ordered_sum<f32x4>(
                splits, [&](int s) { return *(const f32x4*)(src + (size_t)s * slice + n); });
#pragma unroll
            for (int e = 0; e < 4; ++e) x[e] = v[e];
        } else {
            x[0] = ordered_sum<float>(splits, [&](int s) { return src[(size_t)s * slice + n]; });
        }
        float y[VEC];
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            y[e] = activate_dyn(x[e] + add[e], act);
            rs += y[e];
        }
        if constexpr (VEC == 4) {
            if constexpr (OUT_BF16) {
                u32x2 pk = {pack_bf16x2(y[0], y[1]), pack_bf16x2(y[2], y[3])};
                *(u32x2*)((unsigned short*)C + out + n) = pk;
            } else {
                f32x4 o = {y[0], y[1], y[2], y[3]};
                *(f32x4*)((float*)C + out + n) = o;
            }
        } else {
            if constexpr (OUT_BF16) ((unsigned short*)C)[out + n] = (unsigned short)(pack_bf16x2(y[0], 0.0f) & 0xffffu);
            else ((float*)C)[out + n] = y[0];
        }
    }
    if (rowsum) {
        // fixed butterfly over the 64 lanes
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) rs += __shfl_xor(rs, off);
        if (lane == 0) {
            if (nseg == 1) rowsum[row] = rs;
            else rs_part[(b * nseg + seg) * (size_t)M + m] = rs;
        }
    }
}

int splitk_reduce_segments(int M, int N, int batch)
{
    // about 4096 waves, segments of whole 256-column trips
    const long long rows = (long long)M * batch;
    long long want = (4096 + rows - 1) / rows;
    const long long most = (N + 255) / 256;
    if (want > most) want = most;
    if (want < 1) want = 1;
    const long long cols = (((N + want - 1) / want) + 255) / 256 * 256;
    return (int)((N + cols - 1) / cols);
}

hipError_t launch_splitk_reduce(const float* ws, const float* bias, void* C, float* rowsum, float* rs_part,
                                int nseg, int M, int N, int batch, int splits, int act, int dtype, hipStream_t s)
{
    const size_t rows = (size_t)M * batch;
    const size_t blocks = (rows + 3) / 4;
    if (blocks == 0 || blocks > 0x7fffffffULL || nseg < 1 || nseg > 65535) return hipErrorInvalidValue;
    const int seg_cols = (((N + nseg - 1) / nseg) + 255) / 256 * 256;
    const bool vec = (N % 4 == 0) && (((uintptr_t)ws | (uintptr_t)C | (uintptr_t)bias) % 16 == 0);
    const dim3 g((unsigned int)blocks, (unsigned int)nseg), t(256);
#define PGK_RED(V, BF) hipLaunchKernelGGL((splitk_reduce_kernel<V, BF>), g, t, 0, s, ws, bias, C, rowsum, rs_part, seg_cols, M, N, batch, splits, act)
    if (dtype == DT_BF16) { if (vec) PGK_RED(4, true); else PGK_RED(1, true); }
    else { if (vec) PGK_RED(4, false); else PGK_RED(1, false); }
#undef PGK_RED
    return hipGetLastError();
}

}  // namespace pgk
