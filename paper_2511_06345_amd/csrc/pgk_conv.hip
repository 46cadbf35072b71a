// Helpers of the one-dimensional convolution (PRAGMA's second case study, Section 4.4
// "Conv Standard 1D"; the operator is the usual cross-correlation with zero padding).
// The convolution itself runs in the GEMM kernels: with stride 1,
//     y[b] (Cout x Lout) = sum over taps k of  W_k (Cout x Cin)  *  x[b] shifted by k * dilation - pad,
// so a K loop that walks tap after tap over the input channels reads, for each K tile, a plain
// sub-block of the padded input as its B operand.  What is needed beside that:
//   * conv_pad_input: the input with `pad` zeros in front of every row and zeros after it
//     up to a row length that keeps rows 16-byte aligned (skipped when there is no padding
//     and the rows are aligned already);
//   * conv_repack_weights: w[Cout][Cin][Kw] -> w'[Cout][Kw][Cin], so that the K index runs
//     over the channels inside a tap;
//   * conv_prepare: the regrouped weights together with the zero-padded strips that the tile
//     columns at the ends of the rows read when the input is used in place.
// All are streaming copies.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "pgk_device.h"
#include "pgk_kernels.h"

namespace pgk {

namespace {

template <typename T>
__global__ __launch_bounds__(256) void conv_pad_input_kernel(const T* __restrict__ x, T* __restrict__ xp,
                                                             long long rows, int L, int Lp, int pad)
{
    // one workgroup row-slab: blockIdx.y = row (batch entry x channel), blockIdx.x = slab of 1024 outputs
    const long long row = blockIdx.y;
    if (row >= rows) return;
    const int j0 = blockIdx.x * 1024 + threadIdx.x;
    const T* src = x + (size_t)row * (size_t)L;
    T* dst = xp + (size_t)row * (size_t)Lp;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int j = j0 + 256 * u;
        if (j < Lp) {
            const int s = j - pad;
            dst[j] = (s >= 0 && s < L) ? src[s] : T(0);
        }
    }
}

struct EdgeCols { int first[3]; };

template <typename T>
__global__ __launch_bounds__(256) void conv_repack_weights_kernel(const T* __restrict__ w, T* __restrict__ wr,
                                                                  int Cout, int Cin, int Cin_pad, int Kw)
{
    const long long total = (long long)Cout * Cin_pad * Kw;
    const long long t = (long long)blockIdx.x * 256 + threadIdx.x;     // index into wr: (co, k, ci)
    if (t >= total) return;
    const int ci = (int)(t % Cin_pad);
    const long long r = t / Cin_pad;
    const int k = (int)(r % Kw);
    const long long co = r / Kw;
    wr[t] = ci < Cin ? w[(co * Cin + ci) * Kw + k] : T(0);
}

// One 16-byte chunk of the regrouped weights: wr[co][k][ci0 .. ci0 + EPC) = w[co][ci][k] for ci < Cin,
// 0 for the padding channels up to Cin_pad (a multiple of the chunk).  c: chunk index (co, k, ci / EPC).
template <typename T>
__device__ __forceinline__ void repack_weight_chunk(long long c, const T* __restrict__ w, T* __restrict__ wr,
                                                    int Cout, int Cin, int Cin_pad, int Kw)
{
    constexpr int EPC = 16 / (int)sizeof(T);
    const int cpr = Cin_pad / EPC;
    if (c >= (long long)Cout * Kw * cpr) return;
    const int ci0 = (int)(c % cpr) * EPC;
    const long long q = c / cpr;
    const int k = (int)(q % Kw);
    const long long co = q / Kw;
    T v[EPC];
#pragma unroll
    for (int u = 0; u < EPC; ++u) v[u] = ci0 + u < Cin ? w[(co * Cin + ci0 + u) * Kw + k] : T(0);
    u32x4 out;
    __builtin_memcpy(&out, v, 16);
    *(u32x4*)(wr + (size_t)c * EPC) = out;
}

// xc[c][b][ci][j] = x[b][ci][(j + h) * stride + phase - pad] (inside [0, L), ci < Cin; else 0) with
// c = phase * shifts + h.  Bound by its traffic (the input once, the copies once).  A thread makes the
// 16-byte chunk at one (row, j) of all stride * shifts copies, from one run of the input: for STRIDE 1
// and 2, where that run lies inside the row, with 16-byte loads from any element on; else (STRIDE 0:
// any other stride, and at the ends of rows) element by element.  bf16 [8, 512, 4096], two shifted copies:
// 36 us with a thread per chunk of one copy and element loads, 20 so.  Large strides make few such threads with much
// to do each: then `groups` of workgroups share the phases (see launch_conv_phase_copies).  Also regroups the weights (padded
// to Cin_pad channels) into wr.
template <typename T, int STRIDE, int SHIFTS>
__global__ __launch_bounds__(256) void conv_phase_copies_kernel(const T* __restrict__ x, T* __restrict__ xc, unsigned int rows,
                                                                int Cin, int Cin_pad, int L, int Lq, int pad, int stride_any,
                                                                unsigned int copy_blocks, int groups,
                                                                const T* __restrict__ w, T* __restrict__ wr, int Cout, int Kw)
{
    constexpr int EPC = 16 / (int)sizeof(T);
    // the workgroups after the copies regroup the weights (same launch: a second one costs as much
    // as either piece of work)
    if (blockIdx.x >= copy_blocks * groups) {
        repack_weight_chunk<T>((long long)(blockIdx.x - copy_blocks * groups) * 256 + threadIdx.x, w, wr, Cout, Cin, Cin_pad, Kw);
        return;
    }
    const int stride = STRIDE > 0 ? STRIDE : stride_any;
    // the phases of this workgroup
    const int group = STRIDE > 0 ? 0 : (int)(blockIdx.x / copy_blocks), block = STRIDE > 0 ? (int)blockIdx.x : (int)(blockIdx.x % copy_blocks);
    const int per = STRIDE > 0 ? STRIDE : (stride + groups - 1) / groups;
    const int p0 = group * per, p1 = p0 + per < stride ? p0 + per : stride;
    const unsigned int cpr = (unsigned int)(Lq / EPC);        // chunks per row
    const unsigned long long chunk0 = (unsigned long long)block * 256u;
    const unsigned int row0 = (unsigned int)(chunk0 / cpr), in0 = (unsigned int)(chunk0 - (unsigned long long)row0 * cpr) + threadIdx.x;
    const unsigned int row = row0 + in0 / cpr;                // b * Cin_pad + ci
    if (row >= rows) return;
    const int j0 = (int)(in0 % cpr) * EPC;
    const unsigned int b = row / (unsigned int)Cin_pad;
    const int ci = (int)(row - b * (unsigned int)Cin_pad);
    T* dst = xc + (size_t)row * (size_t)Lq + j0;
    const size_t plane = (size_t)rows * (size_t)Lq;           // elements of one copy
    const T* src = x + ((size_t)b * (size_t)Cin + (size_t)(ci < Cin ? ci : 0)) * (size_t)L;
    const long long s0 = (long long)j0 * stride - pad;        // where the run starts
    if constexpr (STRIDE > 0) {
        constexpr int RUN = (EPC + SHIFTS - 1) * STRIDE;      // ... and its elements
        if (ci < Cin && s0 >= 0 && s0 + RUN <= L) {
            T v[RUN];
            using chunk_at_element = typename std::conditional<sizeof(T) == 2, u32x4_align2, u32x4_align4>::type;
#pragma unroll
            for (int q = 0; q < STRIDE; ++q) {
                const u32x4 c = *(const chunk_at_element*)(src + s0 + q * EPC);
                __builtin_memcpy(v + q * EPC, &c, 16);
            }
#pragma unroll
            for (int e = EPC * STRIDE; e < RUN; ++e) v[e] = src[s0 + e];
#pragma unroll
            for (int p = 0; p < STRIDE; ++p)
#pragma unroll
                for (int h = 0; h < SHIFTS; ++h) {
                    T o[EPC];
#pragma unroll
                    for (int e = 0; e < EPC; ++e) o[e] = v[(e + h) * STRIDE + p];
                    u32x4 out;
                    __builtin_memcpy(&out, o, 16);
                    *(u32x4*)(dst + (size_t)(p * SHIFTS + h) * plane) = out;
                }
            return;
        }
    }
    for (int p = p0; p < p1; ++p)
#pragma unroll
        for (int h = 0; h < SHIFTS; ++h) {
            T v[EPC];
#pragma unroll
            for (int e = 0; e < EPC; ++e) {
                const long long s = s0 + (long long)(e + h) * stride + p;
                v[e] = (ci < Cin && s >= 0 && s < L) ? src[s] : T(0);
            }
            u32x4 out;
            __builtin_memcpy(&out, v, 16);
            *(u32x4*)(dst + (size_t)(p * SHIFTS + h) * plane) = out;
        }
}

// Both preparations of the in-place path in one launch (each is a few microseconds of work;
// a second launch costs as much again).  One thread per 16-byte chunk of output: threads
// [0, strip_chunks) fill the strips, strips[e][row][j] = x[row][first[e] + j] inside [0, L), else
// 0 (W, the strip's row length, is a multiple of the chunk), numbered (chunk of the row, row,
// edge) with the chunk fastest; the rest regroup the weights, wr[co][k][ci] = w[co][ci][k], eight
// (bf16) or four (fp32) consecutive ci per thread (Cin is a multiple of the chunk on this path).
template <typename T>
__global__ __launch_bounds__(256) void conv_prepare_kernel(const T* __restrict__ x, T* __restrict__ strips, long long rows,
                                                           int L, int W, EdgeCols cols, long long strip_chunks,
                                                           const T* __restrict__ w, T* __restrict__ wr, int Cout, int Cin, int Kw)
{
    constexpr int EPC = 16 / (int)sizeof(T);
    const long long t = (long long)blockIdx.x * 256 + threadIdx.x;
    T v[EPC];
    T* dst;
    if (t < strip_chunks) {
        const int cpr = W / EPC;                              // chunks per strip row
        const long long r = t / cpr;
        const int j0 = (int)(t - r * cpr) * EPC;
        const long long row = r % rows;
        const int e = (int)(r / rows);
        const T* src = x + (size_t)row * (size_t)L;
        const long long s0 = (long long)cols.first[e] + j0;
#pragma unroll
        for (int u = 0; u < EPC; ++u) {
            const long long sidx = s0 + u;
            v[u] = (sidx >= 0 && sidx < L) ? src[sidx] : T(0);
        }
        dst = strips + ((size_t)e * (size_t)rows + (size_t)row) * (size_t)W + j0;
    } else {
        repack_weight_chunk<T>(t - strip_chunks, w, wr, Cout, Cin, Cin, Kw);
        return;
    }
    u32x4 out;
    __builtin_memcpy(&out, v, 16);
    *(u32x4*)dst = out;
}

}  // namespace

hipError_t launch_conv_prepare(const void* x, void* strips, long long rows, int L, int W, int n_edges, const int* first_col,
                               const void* w, void* wr, int Cout, int Cin, int Kw, int dtype, hipStream_t s)
{
    const int epc = dtype == DT_BF16 ? 8 : 4;
    if (rows <= 0 || n_edges < 0 || n_edges > 3) return hipErrorInvalidValue;
    // whole 16-byte chunks on both sides (the callers' plan guarantees it), 16-byte aligned buffers
    if (Cin % epc != 0 || (n_edges > 0 && W % epc != 0)) return hipErrorInvalidValue;
    if (((uintptr_t)strips | (uintptr_t)wr) % 16 != 0) return hipErrorInvalidValue;
    EdgeCols cols{};
    for (int e = 0; e < n_edges; ++e) cols.first[e] = first_col[e];
    const long long strip_chunks = n_edges > 0 ? (long long)(W / epc) * rows * n_edges : 0;
    const long long repack_chunks = (long long)Cout * Kw * (Cin / epc);
    const long long blocks = (strip_chunks + repack_chunks + 255) / 256;
    if (blocks <= 0 || blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    if (dtype == DT_BF16)
        hipLaunchKernelGGL(conv_prepare_kernel<unsigned short>, dim3((unsigned int)blocks), dim3(256), 0, s,
                           (const unsigned short*)x, (unsigned short*)strips, rows, L, W, cols, strip_chunks,
                           (const unsigned short*)w, (unsigned short*)wr, Cout, Cin, Kw);
    else
        hipLaunchKernelGGL(conv_prepare_kernel<float>, dim3((unsigned int)blocks), dim3(256), 0, s, (const float*)x,
                           (float*)strips, rows, L, W, cols, strip_chunks, (const float*)w, (float*)wr, Cout, Cin, Kw);
    return hipGetLastError();
}

hipError_t launch_conv_phase_copies(const void* x, void* xc, long long B, int Cin, int Cin_pad, int L, int Lq, int pad,
                                    int stride, int shifts, const void* w, void* wr, int Cout, int Kw, int dtype, hipStream_t s)
{
    const int epc = dtype == DT_BF16 ? 8 : 4;
    if (Lq % epc != 0 || Cin_pad % epc != 0 || B <= 0) return hipErrorInvalidValue;
    if (((uintptr_t)xc | (uintptr_t)wr) % 16 != 0) return hipErrorInvalidValue;
    if (shifts < 1 || shifts > 2 || (shifts == 2 && dtype != DT_BF16)) return hipErrorInvalidValue;
    const long long rows = B * (long long)Cin_pad, chunks = rows * (Lq / epc);
    const long long copy_blocks = (chunks + 255) / 256;
    const long long repack_chunks = (long long)Cout * Kw * (Cin_pad / epc);
    // Phases of one position lie side by side, so a thread that makes all of them reads its lines once -- if its
    // wave's (stride KiB) survive in the caches until the last phase and there are enough such threads.  us per call,
    // one group per phase / all phases in a thread:
    //   up to 32: [8, 64, 16000] * [128, 64, 32] stride 16 fp32 118 / 89 (500 workgroups), bf16 85 / 72 (250), batch 1 bf16
    //     33 / 56 (31), fp32 47 / 50 and 44 with four groups (62): groups until every CU has a workgroup;
    //   up to 8 less is shared, and what counts is that loads are in flight everywhere: groups until there are 2048 or 4096
    //     workgroups, in bf16 up to 4 one per phase.  11800 shapes of strides 3 to 8, share that is more than 5 % slower than with one per phase
    //     and mean gain over it: fp32 with 512 workgroups as the aim 3.9 % and 1.09, with 4096 1.5 % and 1.09, bf16 14.3 % and 1.005, and
    //     3.7 % and 1.02 (bf16 [9, 35, 4921] stride 4 17.9 us, with all phases in a thread 25.5);
    //   up to 64: [16, 64, 16000] stride 48 fp32 336 / 211 (333), [1, 128, 64000] stride 64 bf16 184 / 114 (62), [1, 64, 16000] stride
    //     48 fp32 48 / 75 (20); anything between one group and all of them is slower than the better one;
    //   above: [16, 64, 19000] stride 65 bf16 125 / 257 (146), [1, 64, 48000] stride 160 fp32 62 / 151 (18), bf16 39 / 203 (9); the other
    //     way round in bf16 with [8, 64, 48000] stride 160 (375 / 298).
    const long long enough = stride > 8 ? 256 : dtype == DT_BF16 || stride <= 4 ? 4096 : 2048;
    const long long groups = stride <= 2                                          ? 1
                             : (dtype == DT_BF16 && stride <= 4) || stride > 64 ? stride
                             : stride <= 32 ? std::max<long long>(1, std::min<long long>(stride, enough / copy_blocks))
                                            : (copy_blocks >= 48 ? 1 : stride);
    const long long blocks = copy_blocks * groups + (repack_chunks + 255) / 256;
    if (rows > 0xffffffffLL || blocks <= 0 || blocks > 0x7fffffffLL) return hipErrorInvalidValue;
#define PGK_COPIES(T, ST, SH)                                                                                            \
    hipLaunchKernelGGL((conv_phase_copies_kernel<T, ST, SH>), dim3((unsigned int)blocks), dim3(256), 0, s, (const T*)x, (T*)xc, \
                       (unsigned int)rows, Cin, Cin_pad, L, Lq, pad, stride, (unsigned int)copy_blocks, (int)groups, (const T*)w, (T*)wr, Cout, Kw)
    if (dtype == DT_BF16) {
        if (shifts == 2) { if (stride == 1) PGK_COPIES(unsigned short, 1, 2); else if (stride == 2) PGK_COPIES(unsigned short, 2, 2); else PGK_COPIES(unsigned short, 0, 2); }
        else { if (stride == 1) PGK_COPIES(unsigned short, 1, 1); else if (stride == 2) PGK_COPIES(unsigned short, 2, 1); else PGK_COPIES(unsigned short, 0, 1); }
    } else {
        if (stride == 1) PGK_COPIES(float, 1, 1); else if (stride == 2) PGK_COPIES(float, 2, 1); else PGK_COPIES(float, 0, 1);
    }
#undef PGK_COPIES
    return hipGetLastError();
}

hipError_t launch_conv_pad_input(const void* x, void* xp, long long rows, int L, int Lp, int pad, int dtype, hipStream_t s)
{
    if (rows <= 0 || rows > 65535LL * 65535LL) return hipErrorInvalidValue;
    // grid.y is limited to 65535: fold the rows when there are more
    const unsigned int slabs = (unsigned int)((Lp + 1023) / 1024);
    for (long long r0 = 0; r0 < rows; r0 += 65535) {
        const long long n = rows - r0 < 65535 ? rows - r0 : 65535;
        const dim3 grid(slabs, (unsigned int)n);
        if (dtype == DT_BF16)
            hipLaunchKernelGGL(conv_pad_input_kernel<unsigned short>, grid, dim3(256), 0, s,
                               (const unsigned short*)x + (size_t)r0 * L, (unsigned short*)xp + (size_t)r0 * Lp, n, L, Lp, pad);
        else
            hipLaunchKernelGGL(conv_pad_input_kernel<float>, grid, dim3(256), 0, s,
                               (const float*)x + (size_t)r0 * L, (float*)xp + (size_t)r0 * Lp, n, L, Lp, pad);
    }
    return hipGetLastError();
}

hipError_t launch_conv_repack_weights(const void* w, void* wr, int Cout, int Cin, int Cin_pad, int Kw, int dtype, hipStream_t s)
{
    const long long total = (long long)Cout * Cin_pad * Kw;
    const long long blocks = (total + 255) / 256;
    if (blocks <= 0 || blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    if (dtype == DT_BF16)
        hipLaunchKernelGGL(conv_repack_weights_kernel<unsigned short>, dim3((unsigned int)blocks), dim3(256), 0, s,
                           (const unsigned short*)w, (unsigned short*)wr, Cout, Cin, Cin_pad, Kw);
    else
        hipLaunchKernelGGL(conv_repack_weights_kernel<float>, dim3((unsigned int)blocks), dim3(256), 0, s,
                           (const float*)w, (float*)wr, Cout, Cin, Cin_pad, Kw);
    return hipGetLastError();
}

}  // namespace pgk
