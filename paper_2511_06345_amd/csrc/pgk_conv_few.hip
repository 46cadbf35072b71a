// One-dimensional convolution with few input channels (the first layer over a waveform, RGB-like
// inputs): K = Cin * Kw is a handful to a few hundred, so the convolution is bound by writing its
// output -- [8, 1, 160000] * [512, 1, 10], stride 5, fp32: 524 MB of output, 102 us at a copy's 5.1 TB/s, from 5 MB
// of input -- and next by the activation (GELU: sixteen operation slots per output, about 50 us of
// the vector ALUs); the products, on the fp32 matrix instruction, take 20 us of another pipe.
// Same operator as pgk_conv1d (PRAGMA Section 4.4 names the task).
//
// How: a workgroup of four waves owns up to 512 output positions (tiles of 128) and a range of output
// channels.  The input of its positions (as fp32, zeros outside the row) and the weights of its
// channels, k-major, go into LDS once; then every wave takes blocks of 32 channels, tile after tile,
// with no barrier any more.
// Channels are the rows and positions the columns of the 32 x 32 x 2 instruction, column j of block q
// standing for position 4 j + q: a lane's four accumulators of one channel are then four neighbouring
// positions, and a store instruction writes two runs of 512 contiguous bytes (bf16: 256) straight from
// the registers.
// Rows of any length: stores off their natural alignment cost twice their requests to L2 (fp32, Lout 32000
// 116 us, 31999 184 with stores aligned to 16 bytes only).  So a block of channels is not 32 neighbours
// but every fourth or sixteenth channel (`every`): their rows all start at the same offset modulo as many
// elements, and the wave moves its window of positions to the left by that offset.
#include <hip/hip_runtime.h>

#include "pgk_device.h"
#include "pgk_kernels.h"

namespace pgk {

namespace {

constexpr int kTilePos = 128;                   // output positions of a tile
constexpr int kMaxLdsFloats = 20 * 1024;        // 80 KiB: at least two workgroups per CU

struct FewArgs {
    const void* x;
    const void* w;
    const float* bias;
    void* y;
    int Cin, L, Cout, Kw, stride, pad, dil, Lout;
    int K, K2;               // Cin * Kw, and rounded up to a whole pair
    int ch, ch_stride;       // channels per workgroup (a multiple of 128), floats between LDS weight rows
    int slab;                // input positions per channel in LDS
    int tiles;               // position tiles per workgroup
    int every;               // 4 or 16: a block of channels is every fourth or sixteenth
    int groups, chunks;      // workgroups along a row, channel ranges
};

constexpr int kInFlight = 8;                    // loads per thread that the copies into LDS keep in flight

template <bool BF16>
__device__ __forceinline__ float element(const void* base, size_t i)
{
    if constexpr (BF16) return bf16_bits_to_float(((const unsigned short*)base)[i]);
    else return ((const float*)base)[i];
}

// where channel c of the range lies in LDS: the 32 channels of a block side by side
__device__ __forceinline__ int channel_slot(int c, int every)
{
    const int in = c & (32 * every - 1);
    return (c - in) + (in & (every - 1)) * 32 + in / every;
}

// STEPS > 0: Cin * Kw of at most 2 STEPS, weights of a block in registers for all its tiles.
// STREAM: non-temporal stores.  With every sixteenth channel a row's runs are whole 64-byte pieces, and past L2 they go
// out faster ([8, 1, 160000] * [512, 1, 10], stride 5: 137 us with plain stores, 116 so); with every fourth a run starts on any 16
// bytes and L2 has to put lines together (15999 positions of 2 channels 64 us with plain stores, 109 so); rows on
// the 64-byte grid are even (32000 positions 109 and 111, bf16 120000 53 and 58, 64 channels of 160000 77 and 69).  For outputs beyond
// what the last-level cache of 256 MiB takes only, which plain stores end in: 13 x 384 rows of 13325 (266 MB) 51 us with plain stores, 61 so,
// 14 x 384 of 7188 (155 MB) 34 and 41; 9 x 320 of 27050 (312 MB) 89 and 81, 15 x 320 of 24766 (476 MB) 131 and 105.
template <bool BF16, int ACT, int STEPS, bool STREAM = false>
__global__ __launch_bounds__(256, 4) void conv_few_channels_kernel(const FewArgs p)
{
#if defined(__HIP_DEVICE_COMPILE__)
    // the weights [K2][ch_stride], the biases [ch] (16-byte aligned), where k lies in the input [K2], the input
    extern __shared__ __attribute__((aligned(16))) float lds[];
    float* const wt = lds;
    float* const bias = wt + p.K2 * p.ch_stride;
    int* const k_at = (int*)(bias + p.ch);
    float* const in = (float*)(k_at + p.K2);

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, half = lane >> 5;
    unsigned int u = blockIdx.x;
    const int group = (int)(u % (unsigned int)p.groups); u /= (unsigned int)p.groups;
    const int chunk = (int)(u % (unsigned int)p.chunks);
    const size_t b = u / (unsigned int)p.chunks;
    const int c0 = chunk * p.ch;
    const int n_ch = p.Cout - c0 < p.ch ? p.Cout - c0 : p.ch;          // channels of this workgroup that exist
    const int l0 = group * p.tiles * kTilePos;                         // its first position

    // the input (up to every - 1 positions early, for the shifted windows), channel-major
    const int n_in = p.Cin * p.slab;
    const long long first = ((long long)l0 - (p.every - 1)) * p.stride - p.pad;
    for (int i0 = tid; i0 < n_in; i0 += 256 * kInFlight) {
        float v[kInFlight];
#pragma unroll
        for (int q = 0; q < kInFlight; ++q) {
            const int i = i0 + 256 * q, ci = i / p.slab;
            const long long at = first + (i - ci * p.slab);
            v[q] = (i < n_in && at >= 0 && at < p.L) ? element<BF16>(p.x, (b * p.Cin + ci) * (size_t)p.L + (size_t)at) : 0.0f;
        }
#pragma unroll
        for (int q = 0; q < kInFlight; ++q) { const int i = i0 + 256 * q; if (i < n_in) in[i] = v[q]; }
    }
    // the range's weights are contiguous; channels beyond them and the k that only fills up the
    // last pair count as zero
    const int n_w = n_ch * p.K;
    for (int i0 = tid; i0 < n_w; i0 += 256 * kInFlight) {
        float v[kInFlight];
#pragma unroll
        for (int q = 0; q < kInFlight; ++q) { const int i = i0 + 256 * q; v[q] = i < n_w ? element<BF16>(p.w, (size_t)c0 * p.K + i) : 0.0f; }
#pragma unroll
        for (int q = 0; q < kInFlight; ++q) {
            const int i = i0 + 256 * q, co = i / p.K;
            if (i < n_w) wt[(i - co * p.K) * p.ch_stride + channel_slot(co, p.every)] = v[q];
        }
    }
    for (int i = tid; i < p.ch; i += 256) {
        const int at = channel_slot(i, p.every);
        if (i >= n_ch) for (int k = 0; k < p.K; ++k) wt[k * p.ch_stride + at] = 0.0f;
        if (p.K2 > p.K) wt[p.K * p.ch_stride + at] = 0.0f;
        bias[at] = (p.bias && i < n_ch) ? p.bias[c0 + i] : 0.0f;
    }
    for (int k = tid; k < p.K2; k += 256) k_at[k] = k < p.K ? (k / p.Kw) * p.slab + (k % p.Kw) * p.dil : 0;
    __syncthreads();

    // (the k that fills up the last pair: whatever lies in its place must not meet its zero weight)
    const bool odd_k = p.K2 > p.K;
    int at[STEPS > 0 ? STEPS : 1];
    if constexpr (STEPS > 0) {
#pragma unroll
        for (int s = 0; s < STEPS; ++s) at[s] = 2 * s < p.K2 ? k_at[2 * s + half] + 4 * l32 * p.stride : 0;
    }
    constexpr int ES = BF16 ? 2 : 4;
    const size_t row_of_wg = (b * p.Cout + c0) * (size_t)p.Lout;

    // block bl: the channels cb + every i + cls, i < 32
    for (int bl = wave; bl < p.ch / 32; bl += 4) {
        const int cls = bl & (p.every - 1), cb = (bl - cls) * 32, slot0 = bl * 32;
        if (cb + cls >= n_ch) continue;
        // its windows start `shift` positions left of the tiles' starts: its rows' first element lies that
        // many elements behind a multiple of `every`
        const size_t row0 = row_of_wg + (size_t)(cb + cls) * (size_t)p.Lout;
        const int shift = -(int)(((size_t)p.y / ES + row0) & (size_t)(p.every - 1));
        const float* const wk = wt + half * p.ch_stride + slot0 + l32;
        float a[STEPS > 0 ? STEPS : 1];
        if constexpr (STEPS > 0) {
#pragma unroll
            for (int s = 0; s < STEPS; ++s) a[s] = 2 * s < p.K2 ? wk[2 * s * p.ch_stride] : 0.0f;
        }
        // the block's rows: 32-bit offsets from the first (checked on the host)
        auto rows = __builtin_amdgcn_make_buffer_rsrc((unsigned char*)p.y + row0 * ES, 0, (int)0xffffffffu, 0x00020000);
        for (int t = 0; t < p.tiles; ++t) {
            const int pos = l0 + t * kTilePos + shift + 4 * l32;       // the first of this lane's four positions
            const float* const src = in + (t * kTilePos + p.every - 1 + shift) * p.stride;
            f32x16 acc[4];
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[q][e] = 0.0f;
            if constexpr (STEPS > 0) {
#pragma unroll
                for (int s = 0; s < STEPS; ++s) {
                    if (2 * s >= p.K2) break;
                    const bool fill = odd_k && 2 * s + 2 == p.K2 && half == 1;
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const float x = src[at[s] + q * p.stride];
                        acc[q] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[s], fill ? 0.0f : x, acc[q], 0, 0, 0);
                    }
                }
            } else {
#pragma unroll 2
                for (int k = 0; k < p.K2; k += 2) {
                    const float* const from = src + k_at[k + half] + 4 * l32 * p.stride;
                    const float w = wk[k * p.ch_stride];
                    const bool fill = odd_k && k + 2 == p.K2 && half == 1;
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        acc[q] = __builtin_amdgcn_mfma_f32_32x32x2f32(w, fill ? 0.0f : from[q * p.stride], acc[q], 0, 0, 0);
                }
            }
            // register 4 g + e of accumulator q: channel cb + every (8 g + 4 half + e) + cls, position pos + q
            const bool whole = pos >= 0 && pos + 4 <= p.Lout;
            const unsigned int lane_off = (unsigned int)(4 * half * p.every) * (unsigned int)p.Lout * ES + (unsigned int)pos * ES;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                if (cb + 8 * g * p.every + cls >= n_ch) break;
                const f32x4 bc = *(const f32x4*)(bias + slot0 + 8 * g + 4 * half);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    float y[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) y[q] = activate<ACT>(acc[q][4 * g + e] + bc[e]);
                    if (cb + p.every * (8 * g + 4 * half + e) + cls >= n_ch) continue;
                    const unsigned int row_off = (unsigned int)(p.every * (8 * g + e)) * (unsigned int)p.Lout * ES;
                    if constexpr (BF16) {
                        const u32x2 pk = {pack_bf16x2(y[0], y[1]), pack_bf16x2(y[2], y[3])};
                        if (whole) {
                            __builtin_amdgcn_raw_buffer_store_b64(pk, rows, lane_off, row_off, 0);
                        } else {
#pragma unroll
                            for (int q = 0; q < 4; ++q)
                                if (pos + q >= 0 && pos + q < p.Lout)
                                    __builtin_amdgcn_raw_buffer_store_b16((unsigned short)(q % 2 ? pk[q / 2] >> 16 : pk[q / 2] & 0xffffu), rows, lane_off + 2 * q, row_off, 0);
                        }
                    } else {
                        if (whole) {
                            const f32x4 v = {y[0], y[1], y[2], y[3]};
                            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), rows, lane_off, row_off, STREAM ? 2 : 0);
                        } else {
#pragma unroll
                            for (int q = 0; q < 4; ++q)
                                if (pos + q >= 0 && pos + q < p.Lout)
                                    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned int, y[q]), rows, lane_off + 4 * q, row_off, 0);
                        }
                    }
                }
            }
        }
    }
#endif
}

// LDS of a workgroup in floats (64-bit: the caller's sizes are unchecked)
long long slab_of(long long tiles, long long Kw, long long stride, long long dil) { return (tiles * kTilePos + 14) * stride + (Kw - 1) * dil + 1; }
long long lds_floats(long long Cin, long long Kw, long long stride, long long dil, long long tiles, long long ch)
{
    const long long K2 = (Cin * Kw + 1) / 2 * 2;
    return Cin * slab_of(tiles, Kw, stride, dil) + K2 * (ch + 4) + ch + K2;
}

}  // namespace

// Sums of up to 24 products, or up to 48 for at least 128 channels (which fill the blocks), the input of a
// tile and the weights within 80 KiB of LDS, and enough pairs of a tile and 128 channels: 256, for more than 8
// products 384 (bf16 [29, 1, 1260] * [281, 1, 16], stride 4, 261 pairs: 15.5 us here, 11.3 on the bounds-checked kernel), for the
// longer sums 1024 (bf16 [2, 4, 87346] * [128, 4, 7], 274 pairs: 18 us there, 21 here); with less to do the bounds-checked
// kernel's smaller tiles spread further ([4, 12, 9000] * [128, 12, 7], stride 5: 19 us there, 29 here), and longer sums are its
// strength on few channels ([4, 15, 20000] * [64, 15, 5]: 20 against 28).  Cin * stride input values are copied into
// LDS per position, element by element, and have to be shared by enough channels: not more than 32 of them, nor than
// half the channels plus 4 (bf16 [5, 12, 67038] * [178, 12, 3], stride 5: 69 us here, 42 there; [24, 12, 106417] * [18, 12, 1], stride
// 5: 110 and 43).  Rows of fewer than 64 outputs would leave half a tile empty.
// Of 22500 shapes within the other limits the lines at 384 pairs, 32 values and half the channels take out 2760
// (1300 slower here, 970 faster); 1.4 % of the rest are more than 5 % slower here than there, 6 % without these lines.
bool conv_few_channels_fits(long long B, long long Cin, long long Cout, long long Kw, long long stride, long long dil, long long Lout)
{
    if (Lout < 64 || Cin > 48 || Kw > 48 || stride > 4096 || dil > 4096) return false;
    const long long K = Cin * Kw, units = (Lout + kTilePos - 1) / kTilePos * ((Cout + 127) / 128);
    if (K > 48 || (K > 24 && Cout < 128) || (long double)units * B < (K > 24 ? 1024.0L : K > 8 ? 384.0L : 256.0L)) return false;
    if (Cin * stride > 32 || Cin * stride > Cout / 2 + 4) return false;
    if (Lout * 4 * 128 >= (1LL << 32)) return false;          // a block's 32-bit offsets
    return lds_floats(Cin, Kw, stride, dil, 1, 128) <= kMaxLdsFloats;
}

namespace {
// (non-temporal stores: every sixteenth channel, which is fp32 with at most 16 products only)
template <bool BF16, int ACT>
void launch_few(const FewArgs& a, bool stream, dim3 grid, size_t lds, hipStream_t s)
{
    const dim3 block(256);
    if constexpr (!BF16)
        if (stream) {
            if (a.K2 <= 8) hipLaunchKernelGGL((conv_few_channels_kernel<BF16, ACT, 4, true>), grid, block, lds, s, a);
            else hipLaunchKernelGGL((conv_few_channels_kernel<BF16, ACT, 8, true>), grid, block, lds, s, a);
            return;
        }
    if (a.K2 <= 8) hipLaunchKernelGGL((conv_few_channels_kernel<BF16, ACT, 4>), grid, block, lds, s, a);
    else if (a.K2 <= 16) hipLaunchKernelGGL((conv_few_channels_kernel<BF16, ACT, 8>), grid, block, lds, s, a);
    else hipLaunchKernelGGL((conv_few_channels_kernel<BF16, ACT, 0>), grid, block, lds, s, a);
}
}  // namespace

hipError_t launch_conv_few_channels(const void* x, const void* w, const float* bias, void* y, long long B, int Cin, int L, int Cout,
                                    int Kw, int stride, int pad, int dil, int Lout, int act, int dtype, hipStream_t s)
{
    if (!conv_few_channels_fits(B, Cin, Cout, Kw, stride, dil, Lout)) return hipErrorInvalidValue;
    FewArgs a{};
    a.x = x; a.w = w; a.bias = bias; a.y = y;
    a.Cin = Cin; a.L = L; a.Cout = Cout; a.Kw = Kw; a.stride = stride; a.pad = pad; a.dil = dil; a.Lout = Lout;
    a.K = Cin * Kw;
    a.K2 = (a.K + 1) / 2 * 2;
    // As many channels and up to four tiles as a quarter of a CU's LDS holds, fewer while there are fewer
    // than four workgroups per CU (windows start up to fifteen positions early).
    // Every sixteenth channel: fp32 rows that do not start on 64-byte boundaries, where there are enough
    // channels to fill half of such a block, the products do not weigh and two workgroups per CU are left
    // (8 x 512 rows of 31999: 184 -> 145 us, 116 with non-temporal stores; 300 rows of 14747, 116 workgroups: 15 -> 20 us).  bf16 stores are
    // 8 bytes a lane, and 31999 positions as fast as 32000 with every fourth (84 us).
    const long long es = dtype == DT_BF16 ? 2 : 4;
    const bool rows_aligned = (Lout * es) % 64 == 0 && (reinterpret_cast<uintptr_t>(y) % 64) == 0;
    const bool sixteenth = dtype == DT_F32 && !rows_aligned && Cout >= 256 && a.K2 <= 16 && (long long)Lout * 4 * 512 < (1LL << 32) &&
                           (Lout / kTilePos) * ((Cout + 511LL) / 512) * B >= 512;
    a.every = sixteenth ? 16 : 4;
    const long long unit = 32LL * a.every;
    const long long row_tiles = ((long long)Lout + a.every - 1 + kTilePos - 1) / kTilePos, budget = 10 * 1024;
    long long ch = ((long long)Cout + unit - 1) / unit * unit, tiles = row_tiles < 4 ? row_tiles : 4;
    auto wgs_of = [&]() { return (row_tiles + tiles - 1) / tiles * ((Cout + ch - 1) / ch) * B; };
    while (ch > unit && (lds_floats(Cin, Kw, stride, dil, 1, ch) > budget || wgs_of() < 1024)) ch -= unit;
    while (tiles > 1 && (lds_floats(Cin, Kw, stride, dil, tiles, ch) > budget || wgs_of() < 1024)) --tiles;
    if (lds_floats(Cin, Kw, stride, dil, tiles, ch) > kMaxLdsFloats) { a.every = 4; ch = 128; tiles = 1; }
    a.ch = (int)ch;
    a.tiles = (int)tiles;
    a.ch_stride = a.ch + 4;                              // (the two halves of a wave read neighbouring rows)
    a.slab = (int)slab_of(tiles, Kw, stride, dil);
    a.groups = (int)((row_tiles + tiles - 1) / tiles);
    a.chunks = (int)((Cout + ch - 1) / ch);
    const long long wgs = wgs_of();
    if (wgs <= 0 || wgs > 0x7fffffffLL) return hipErrorInvalidValue;
    const size_t lds = (size_t)lds_floats(Cin, Kw, stride, dil, tiles, ch) * sizeof(float);
    const dim3 grid((unsigned int)wgs);
    const bool stream = a.every == 16 && (long double)B * Cout * Lout * es > 300.0e6L;
#define PGK_FEW_ACT(BF)                                                      \
    switch (act) {                                                           \
    case ACT_RELU: launch_few<BF, ACT_RELU>(a, stream, grid, lds, s); break;         \
    case ACT_GELU_TANH: launch_few<BF, ACT_GELU_TANH>(a, stream, grid, lds, s); break; \
    case ACT_SILU: launch_few<BF, ACT_SILU>(a, stream, grid, lds, s); break;         \
    default: launch_few<BF, ACT_NONE>(a, stream, grid, lds, s); break;               \
    }
    if (dtype == DT_BF16) { PGK_FEW_ACT(true) } else { PGK_FEW_ACT(false) }
#undef PGK_FEW_ACT
    return hipGetLastError();
}

}  // namespace pgk
