// One-dimensional convolution, bf16, the input read in place (the operator of PRAGMA's second case study, Section 4.4; see pgk_conv.hip).
//
// A workgroup of four waves owns BM output channels (128, 64 or 32) and 128 positions of one batch entry.  It walks the input channels
// in blocks of 32: the positions that the tile's outputs read, halo and all, come from memory once per block and lie in LDS as
// [position][channel], so that every tap of the block -- whatever its offset, stride or dilation -- finds the eight channels that a
// lane of the matrix instruction needs in sixteen aligned bytes.  In the layout of memory, [channel][position], taps at odd offsets
// start on 2-byte boundaries, which neither direct copies nor transposing reads take: that costs shifted copies of the input
// or a loop through registers, and strides and channels off the K tile more copies.  Here there are none, positions past a row's ends and
// channels past the last one enter as zeros, and x is read once instead of once per tap.
//  * A thread loads two neighbouring positions of eight channels (4 bytes each, any element), pairs the channels with byte permutes and
//    writes two sixteen-byte pieces.  At the ends of rows a pair is moved back inside, and shifted or cleared when it is written.
//  * The weights are regrouped to [Cout][Kw][channels, padded with zeros to 32] (a small launch before); a block's are copied straight to LDS.
//  * Blocks alternate between two buffers of both: the next block's loads are in flight under this one's taps, nothing else of a block
//    goes to memory (weights fetched tap by tap waited, in order, for the input's loads: four times as long), and one barrier
//    per block suffices.
//  * LDS: row r (a position, or a channel of the weights of a tap), channel octet o at 128 (r / 2) + 16 ((4 (r % 2) + o) ^ (r / 2 % 8)): eight
//    consecutive rows, or eight with stride 2, of one octet lie in different banks.  Sixteen rows on is a constant number of
//    bytes on, so a tap takes one address.
//  * v_mfma_f32_16x16x32_bf16, accumulators in registers, roles as in pgk_gemm_mfma_kernel.h: a lane holds four consecutive positions of a channel.
// What bounds it and what it measured: see conv_bf16_in_place in pgk_api.hip, where the line to the other ways lies.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <type_traits>

#include "pgk_device.h"
#include "pgk_kernels.h"

namespace pgk {

namespace {

constexpr int kBlock = 32;                 // channels per block
constexpr int kCols = 128;                 // positions per tile
constexpr int kGroups = 3;                 // of 128 rows of LDS, at most
constexpr int kMostLds = 80 * 1024;        // bytes of LDS per workgroup, at most (taps_at_a_time)

struct ConvArgs {
    const unsigned short* x;
    const unsigned short* w;               // [Cout][Kw][cin_pad]
    const float* bias;
    unsigned short* y;
    int Cin, cin_pad, L, Cout, Kw, stride, pad, dil, Lout, act;
    int tiles_m, tiles_n, group_m;
    int rows;                              // positions that a tile reads
    int taps;                              // whose weights are in LDS at a time
};

typedef unsigned int u32_align2 __attribute__((aligned(2)));

__device__ __forceinline__ int lds_at(int row, int octet) { return (row >> 1) * 128 + (((((row & 1) << 2) | octet) ^ ((row >> 1) & 7)) << 4); }

// GROUPS: of 128 positions, as many as the tile reads.  PARTS: the weights of a block do not lie in LDS all at once.  (An instance of its own: with
// one loop for both the case without parts was a quarter slower.)
template <int BM, int GROUPS, bool PARTS>
__global__ __launch_bounds__(256, BM == 128 || (BM == 64 && GROUPS == 3) ? 2 : 3) void conv_bf16_kernel(const ConvArgs p)
{
#if defined(__HIP_DEVICE_COMPILE__)
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
    constexpr int WGM = BM >= 64 ? 2 : 1, WGN = 4 / WGM, WM = BM / WGM, WN = kCols / WGN, TM = WM / 16, TN = WN / 16;
    const unsigned int tiles = (unsigned int)p.tiles_m * (unsigned int)p.tiles_n;
    const unsigned int logical = xcd_remap(blockIdx.x, gridDim.x), b = logical / tiles;
    int tm, tn;
    tile_coords(logical - b * tiles, p.tiles_m, p.tiles_n, p.group_m, tm, tn);
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, grp = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WGN, wn = wave % WGN;
    const int rows = (p.rows + 1) / 2 * 2;
    // LDS: two buffers of the input's rows, two of some taps' weights
    const int x_bytes = rows * 64, w_bytes = p.taps * BM * 64;
    unsigned char* const weight_lds = lds + 2 * x_bytes;
    const int first = tn * kCols * p.stride - p.pad;              // the position of row 0
    const bool ends = first < 0 || first + rows > p.L;

    // ---- the input, memory -> registers: of group m rows 2 lane + 128 m and the next one, the eight channels of this wave's octet.
    // A pair that does not lie inside the row is read from the nearest place that does.
    unsigned int v[GROUPS][8];
    unsigned int at[GROUPS];                                      // (bytes from the row's start)
#pragma unroll
    for (int m = 0; m < GROUPS; ++m) {
        const int wanted = first + 2 * lane + 128 * m;
        at[m] = 2u * (unsigned int)(wanted < 0 ? 0 : wanted > p.L - 2 ? p.L - 2 : wanted);
    }
    const unsigned short* const xb = p.x + (size_t)b * (size_t)p.Cin * (size_t)p.L;
    const unsigned int row_bytes = (unsigned int)p.L * 2u;
    auto load = [&](int block) __attribute__((always_inline)) {
        const int c0 = block * kBlock + 8 * wave;
        // (a channel past the last one: another one, cleared when it is written)
        const unsigned char* const from = (const unsigned char*)xb + (size_t)(c0 < p.Cin ? c0 : 0) * (size_t)row_bytes;
        const int left = c0 < p.Cin ? p.Cin - c0 : 1;
#pragma unroll
        for (int m = 0; m < GROUPS; ++m) {
            if (m < GROUPS - 1 || 2 * lane + 128 * m < rows) {    // (the last group's lanes that are past the tile's positions; lane 0 never is)
#pragma unroll
                for (int e = 0; e < 8; ++e) v[m][e] = *(const u32_align2*)(from + ((e < left ? (unsigned int)e * row_bytes : 0u) + at[m]));
            }
        }
    };
    // ---- registers -> LDS
    auto write = [&](int block, unsigned char* to) __attribute__((always_inline)) {
        const int c0 = block * kBlock + 8 * wave;
        if (c0 + 8 > p.Cin) {
#pragma unroll
            for (int m = 0; m < GROUPS; ++m)
#pragma unroll
                for (int e = 0; e < 8; ++e) v[m][e] = c0 + e < p.Cin ? v[m][e] : 0u;
        }
#pragma unroll
        for (int m = 0; m < GROUPS; ++m) {
            const int r = 2 * lane + 128 * m;
            if (ends) {
                const int off = first + r - (int)(at[m] / 2u);                // 0: inside; -1, 1: half of the pair is; else none of it
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const unsigned int w = v[m][e];
                    v[m][e] = off == 0 ? w : off == -1 ? w << 16 : off == 1 ? w >> 16 : 0u;
                }
            }
            if (r >= rows) continue;
            u32x4 even, odd;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                even[q] = __builtin_amdgcn_perm(v[m][2 * q + 1], v[m][2 * q], 0x05040100u);
                odd[q] = __builtin_amdgcn_perm(v[m][2 * q + 1], v[m][2 * q], 0x07060302u);
            }
            *(__attribute__((address_space(3))) u32x4*)PGK_LDS(to + lds_at(r, wave)) = even;
            *(__attribute__((address_space(3))) u32x4*)PGK_LDS(to + lds_at(r + 1, wave)) = odd;
        }
    };
    // ---- the weights, memory -> LDS: a wave instruction copies sixteen channels of a tap, lane s what belongs at 16 s (see lds_at)
    constexpr int QN = BM / 16, PIECES = QN >= 4 ? QN / 4 : 1, TAP_STEP = QN >= 4 ? 1 : 4 / QN;      // (a wave's pieces of a tap, its taps)
    unsigned int w_off[PIECES];
#pragma unroll
    for (int k = 0; k < PIECES; ++k) {
        const int u = (lane & 7) ^ (lane >> 3);
        const int co = tm * BM + 16 * (wave % QN + 4 * k) + 2 * (lane >> 3) + (u >> 2);      // (channels past the last one: it again; not stored)
        w_off[k] = ((unsigned int)(co < p.Cout ? co : p.Cout - 1) * (unsigned int)p.Kw * (unsigned int)p.cin_pad + 8u * (unsigned int)(u & 3)) * 2u;
    }
    auto copy_weights = [&](int block, int tap0, unsigned char* to) __attribute__((always_inline)) {
        const int n = p.Kw - tap0 < p.taps ? p.Kw - tap0 : p.taps, t0 = QN >= 4 ? 0 : wave / QN;
        auto all = __builtin_amdgcn_make_buffer_rsrc((void*)p.w, 0, (int)0xffffffffu, 0x00020000);
        unsigned char* at = to + (t0 * QN + wave % QN) * 1024;
        unsigned int soff = (unsigned int)((tap0 + t0) * p.cin_pad + block * kBlock) * 2u;
        for (int t = t0; t < n; t += TAP_STEP) {
#pragma unroll
            for (int k = 0; k < PIECES; ++k) __builtin_amdgcn_raw_ptr_buffer_load_lds(all, PGK_LDS(at + k * 4096), 16, w_off[k], soff, 0, 0);
            at += TAP_STEP * QN * 1024;
            soff += (unsigned int)(TAP_STEP * p.cin_pad) * 2u;
        }
    };

    // ---- operands of a tap
    const int a_at = lds_at(wm * WM + l16, grp), row0 = (wn * WN + l16) * p.stride;
    auto fetch_a = [&](const unsigned char* weights, int tap, bf16x8 (&f)[TM]) __attribute__((always_inline)) {
        const unsigned char* const from = weights + tap * (BM * 64) + a_at;
#pragma unroll
        for (int i = 0; i < TM; ++i) f[i] = *(const __attribute__((address_space(3))) bf16x8*)PGK_LDS(from + i * 1024);
    };
    auto fetch_b = [&](const unsigned char* input, int tap, bf16x8 (&f)[TN]) __attribute__((always_inline)) {
        const unsigned char* const from = input + lds_at(row0 + tap * p.dil, grp);
#pragma unroll
        for (int j = 0; j < TN; ++j) f[j] = *(const __attribute__((address_space(3))) bf16x8*)PGK_LDS(from + j * 1024 * p.stride);
    };
    f32x4 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    auto multiply = [&](const bf16x8 (&a)[TM], const bf16x8 (&f)[TN]) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int i = 0; i < TM; ++i) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f[j], a[i], acc[i][j], 0, 0, 0);
    };

    float bias[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int co = tm * BM + wm * WM + 16 * i + l16;
        bias[i] = p.bias && co < p.Cout ? p.bias[co] : 0.0f;
    }

    const int blocks = p.cin_pad / kBlock;
    // some taps of a block in LDS: two a trip, each with the next one's operands on their way
    auto multiply_taps = [&](const unsigned char* input, const unsigned char* weights, int tap0) __attribute__((always_inline)) {
        const int n = p.Kw - tap0 < p.taps ? p.Kw - tap0 : p.taps;
        bf16x8 a0[TM], a1[TM], b0[TN], b1[TN];
        fetch_a(weights, 0, a0);
        fetch_b(input, tap0, b0);
        int t = 0;
        for (; t + 2 <= n; t += 2) {
            fetch_a(weights, t + 1, a1);
            fetch_b(input, tap0 + t + 1, b1);
            multiply(a0, b0);
            if (t + 2 < n) {
                fetch_a(weights, t + 2, a0);
                fetch_b(input, tap0 + t + 2, b0);
            }
            multiply(a1, b1);
        }
        if (t < n) multiply(a0, b0);
    };
    // this wave's copies to LDS are there (behind: the eight loads per group of the input that follow them need not be); the barrier
    // sees to the others'
    auto arrived = [&](bool behind) __attribute__((always_inline)) {
        if (behind) {
            if constexpr (GROUPS == 1) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
            else if constexpr (GROUPS == 2) asm volatile("s_waitcnt vmcnt(16)" ::: "memory");
            else asm volatile("s_waitcnt vmcnt(24)" ::: "memory");
        } else {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        }
        __syncthreads();
    };
    load(0);
    copy_weights(0, 0, weight_lds);
    write(0, lds);
    arrived(false);
    int step = 0;
    for (int block = 0; block < blocks; ++block) {
        const unsigned char* const input = lds + (block & 1) * x_bytes;
        unsigned char* const next_input = lds + ((block + 1) & 1) * x_bytes;
        const bool another = block + 1 < blocks;
        // (what is written to now was last read before the barrier that opened this block, or this part of one)
        if constexpr (!PARTS) {
            if (another) {
                load(block + 1);
                copy_weights(block + 1, 0, weight_lds + ((block + 1) & 1) * w_bytes);
            }
            multiply_taps(input, weight_lds + (block & 1) * w_bytes, 0);
            if (another) {
                write(block + 1, next_input);
                arrived(false);
            }
        } else {
            for (int tap0 = 0; tap0 < p.Kw; tap0 += p.taps, ++step) {
                const bool last = tap0 + p.taps >= p.Kw;
                if (!last || another) copy_weights(last ? block + 1 : block, last ? 0 : tap0 + p.taps, weight_lds + ((step + 1) & 1) * w_bytes);
                __builtin_amdgcn_sched_barrier(0);                // (the input's loads behind the copies, as `arrived` counts them)
                if (tap0 == 0 && another) load(block + 1);
                __builtin_amdgcn_sched_barrier(0);
                multiply_taps(input, weight_lds + (step & 1) * w_bytes, tap0);
                if (last && another) write(block + 1, next_input);
                if (!last || another) arrived(tap0 == 0 && another);
            }
        }
    }
    __syncthreads();                                              // the buffers are the epilogue's now

    // ---- epilogue, per wave: sixteen channels at a time through a piece of LDS that only this wave touches, stored in
    // sixteen-byte chunks of whole row pieces, which may start on any element
    constexpr int ROWB = WN * 2, UNITS = ROWB / 16, CH = 16 * UNITS / 64;
    unsigned char* const piece = lds + wave * (16 * ROWB);
    const int n_left = p.Lout - (tn * kCols + wn * WN);           // positions of this wave's part that exist
    auto finish = [&](auto act) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < TM; ++i) {
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const f32x4 s = acc[i][j];
            const u32x2 h = {pack_bf16x2(activate<decltype(act)::value>(s[0] + bias[i]), activate<decltype(act)::value>(s[1] + bias[i])),
                             pack_bf16x2(activate<decltype(act)::value>(s[2] + bias[i]), activate<decltype(act)::value>(s[3] + bias[i]))};
            const int unit = 2 * j + (grp >> 1);
            *(u32x2*)(piece + l16 * ROWB + ((unit ^ (l16 & (UNITS - 1))) << 4) + (grp & 1) * 8) = h;
        }
        asm volatile("" ::: "memory");
        u32x4 out[CH];
#pragma unroll
        for (int t = 0; t < CH; ++t) {
            const int c = lane + 64 * t, r = c / UNITS, cc = c % UNITS;
            out[t] = *(const u32x4*)(piece + r * ROWB + ((cc ^ (r & (UNITS - 1))) << 4));
        }
        asm volatile("" ::: "memory");
#pragma unroll
        for (int t = 0; t < CH; ++t) {
            const int c = lane + 64 * t, r = c / UNITS, cc = c % UNITS;
            const int co = tm * BM + wm * WM + 16 * i + r, left = n_left - 8 * cc;
            if (co >= p.Cout || left <= 0) continue;
            unsigned short* const to = p.y + ((size_t)b * (size_t)p.Cout + (size_t)co) * (size_t)p.Lout + (size_t)(tn * kCols + wn * WN + 8 * cc);
            if (left >= 8) {
                *(u32x4_align2*)to = out[t];
            } else {
#pragma unroll
                for (int e = 0; e < 7; ++e) {
                    if (e >= left) break;
                    to[e] = (unsigned short)(out[t][e / 2] >> (16 * (e & 1)));
                }
            }
        }
    }
    };
    switch (p.act) {
    case ACT_RELU: finish(std::integral_constant<int, ACT_RELU>{}); break;
    case ACT_GELU_TANH: finish(std::integral_constant<int, ACT_GELU_TANH>{}); break;
    case ACT_SILU: finish(std::integral_constant<int, ACT_SILU>{}); break;
    default: finish(std::integral_constant<int, ACT_NONE>{}); break;
    }
#endif
}

template <int BM, int GROUPS, bool PARTS>
hipError_t launch_tile(const ConvArgs& p, unsigned int wgs, size_t lds, hipStream_t s)
{
    if (lds > 64 * 1024) {
        // More than the runtime grants unasked.  The grant is the kernel's and not the call's, so it is the most that any call takes: a
        // thread with a smaller convolution must not lower it between another one's grant and its launch.  Once per device.
        static std::atomic<unsigned long long> granted{0};
        int device = 0;
        hipError_t e = hipGetDevice(&device);
        if (e != hipSuccess) return e;
        const unsigned long long bit = device < 64 ? 1ull << device : 0;
        if (!(granted.load(std::memory_order_acquire) & bit)) {
            e = hipFuncSetAttribute((const void*)conv_bf16_kernel<BM, GROUPS, PARTS>, hipFuncAttributeMaxDynamicSharedMemorySize, kMostLds);
            if (e != hipSuccess) return e;
            granted.fetch_or(bit, std::memory_order_release);
        }
    }
    hipLaunchKernelGGL((conv_bf16_kernel<BM, GROUPS, PARTS>), dim3(wgs), dim3(256), lds, s, p);
    return hipGetLastError();
}

template <int BM, int GROUPS>
hipError_t launch_groups(const ConvArgs& p, unsigned int wgs, size_t lds, hipStream_t s)
{
    // (one group of positions is a single tap at stride 1, whose weights are one part)
    if constexpr (GROUPS > 1) { if (p.taps < p.Kw) return launch_tile<BM, GROUPS, true>(p, wgs, lds, s); }
    return launch_tile<BM, GROUPS, false>(p, wgs, lds, s);
}

template <int BM>
hipError_t launch_rows(const ConvArgs& p, unsigned int wgs, size_t lds, hipStream_t s)
{
    return p.rows <= 128 ? launch_groups<BM, 1>(p, wgs, lds, s) : p.rows <= 256 ? launch_groups<BM, 2>(p, wgs, lds, s) : launch_groups<BM, 3>(p, wgs, lds, s);
}

}  // namespace

// Weights of all taps at a time where two workgroups (of 32 channels three) then fit a CU, else of parts that do: every part is a
// barrier and a wait for its copies, about 1 us with one workgroup on a CU ([1, 384, 2048] x [240, 384, 3] stride 2, parts of one tap 38 us, all three
// at once 23), and with a single workgroup on a CU nothing covers the rest of a block ([14, 38, 36183] x [247, 38, 10], 64 rows all at
// once 415, in two parts 269).
static int taps_at_a_time(long long Kw, long long positions, int rows)
{
    const long long room = 160 * 1024 / (rows == 32 ? 3 : 2) - 2 * positions * 64;
    const long long most = std::max(1LL, std::min(Kw, room / (2 * rows * 64))), parts = (Kw + most - 1) / most;
    return (int)((Kw + parts - 1) / parts);
}

size_t conv_bf16_lds(long long Kw, long long stride, long long dil, long long L, int rows, int* parts)
{
    if (L < 2 || stride > kGroups || dil > kGroups * 128 || Kw > kGroups * 128) return 0;
    const long long positions = ((Kw - 1) * dil + (kCols - 1) * stride + 1 + 1) / 2 * 2;
    if (positions > kGroups * 128) return 0;
    const long long taps = taps_at_a_time(Kw, positions, rows);
    if (parts) *parts = (int)((Kw + taps - 1) / taps);
    return (size_t)(2 * positions * 64 + 2 * taps * rows * 64);
}

hipError_t launch_conv_bf16(const void* x, const void* wr, const float* bias, void* y, long long B, int Cin, int cin_pad, int L, int Cout,
                            int Kw, int stride, int pad, int dil, int Lout, int rows, int act, hipStream_t s)
{
    const size_t lds = conv_bf16_lds(Kw, stride, dil, L, rows);      // (128 rows of input and more: the epilogue's pieces fit)
    if (!lds || lds > (size_t)kMostLds || cin_pad % kBlock != 0 || cin_pad < Cin || (uintptr_t)wr % 16 != 0) return hipErrorInvalidValue;
    ConvArgs p{};
    p.x = (const unsigned short*)x; p.w = (const unsigned short*)wr; p.bias = bias; p.y = (unsigned short*)y;
    p.Cin = Cin; p.cin_pad = cin_pad; p.L = L; p.Cout = Cout; p.Kw = Kw; p.stride = stride; p.pad = pad; p.dil = dil; p.Lout = Lout; p.act = act;
    p.rows = (Kw - 1) * dil + (kCols - 1) * stride + 1;
    p.taps = taps_at_a_time(Kw, (p.rows + 1) / 2 * 2, rows);
    p.tiles_m = (Cout + rows - 1) / rows;
    p.tiles_n = (Lout + kCols - 1) / kCols;
    p.group_m = p.tiles_m < 8 ? p.tiles_m : 8;
    const long long wgs = (long long)p.tiles_m * p.tiles_n * B;
    // (eight rows as 32-bit byte offsets)
    if (L >= (1 << 27)) return hipErrorInvalidValue;
    // (first positions as 32-bit numbers, the weights as 32-bit byte offsets)
    if (wgs <= 0 || wgs > 0x7fffffffLL || ((long long)p.tiles_n * kCols + kGroups * 128) * stride + pad > 0x7fffffffLL ||
        (long long)Cout * Kw * cin_pad >= (1LL << 31) - 64) return hipErrorInvalidValue;
    switch (rows) {
    case 128: return launch_rows<128>(p, (unsigned int)wgs, lds, s);
    case 64: return launch_rows<64>(p, (unsigned int)wgs, lds, s);
    case 32: return launch_rows<32>(p, (unsigned int)wgs, lds, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace pgk
