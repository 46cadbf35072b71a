// fp32 GEMM on the bf16 matrix cores, with the fused epilogue, for gfx950 (MI355X): the kernel
// template and its configurations.  Same operator, arguments and tile shapes as the kernels of
// pgk_gemm_mfma_kernel.h (C = act(A*B + bias), optional row sums; PRAGMA Sections 1 and 4.2 name
// it, the definition is the textbook one).
//
// What bounds an fp32 GEMM on this chip is the fp32 matrix instruction: 157 TFLOP/s, a sixteenth
// of the bf16 one.  Here every operand value is taken apart into three bf16 values that add up to
// it exactly (x = h + m + l with h = x and m = x - h rounded to bf16, l the rest; the differences are exact in
// fp32), and a product is the sum of six bf16 products (a published way of making wide products of narrow ones):
//     a b = ah bh + (ah bm + am bh) + (ah bl + al bh + am bm) + [am bl + al bm + al bl]
// The bracket is left out.  Of values in [2^e, 2^(e+1)) |m| <= 2^(e-8) and |l| <= 2^(e-17), of either sign: it is
// 2^-24 |a b| at the very worst and 2^-27 of it in the root mean square.  A product with an identity matrix gives the other
// factor exactly.
//
// Rounding.  Inside the bf16 matrix instruction sums are cut off downwards, not rounded to nearest.  Were
// the accumulators kept there, every step would cut six times at the size of the whole sum, in one direction.
// So a step's sums start from zero, the five small products' and the large ones' apart, and the vector ALUs
// add them to the accumulators, rounding to nearest: two roundings per 32 k (the fp32 instruction has
// sixteen), cuts only at the size of a step's own sum, and for a single product nothing but the one rounding of its
// two parts.  These adds are a third of the vector operations: 4096^3 640 us without them, 700 with.
// What is left of the direction of the cuts would still show in a sum over many outputs (the row sums).  So odd rows of A
// and odd columns of B enter with their sign turned and the epilogue turns it back, which costs nothing in
// either place: neighbouring outputs err in opposite directions.
// Measured against 64-bit sums (2048 x 2048 outputs), 2-norm of the error, the fp32 instruction / here:
//   A uniform in [-1, 1), B normal: K = 32 1.03e-7 / 0.37e-7, 256 2.9e-7 / 0.8e-7, 4096 1.15e-6 / 0.29e-6, 16384 2.3e-6 / 0.58e-6;
//   both uniform in [0, 1): 32 8.4e-8 / 4.1e-8, 256 2.2e-7 / 0.6e-7, 4096 8.4e-7 / 2.1e-7; and with A falling by 2^20 along K:
//   4096 6.1e-6 / 0.27e-6; A diagonal: 2.53e-8 / 2.60e-8 (the products left out).
//
// Range.  bf16 has the exponents of fp32, so nothing overflows that fp32 holds, with three
// exceptions, and all are found and made good inside the kernel: the tile is then computed again
// with the fp32 matrix instruction (fallback below).
//  * A value above the largest bf16 (3.39e38) rounds to infinity, and an infinity or NaN among the
//    operands turns into NaN where fp32 would give an infinity.  Either way the accumulators it
//    touches are not finite, so: any accumulator of the tile that is not finite.
//  * The low term of a value below about 2^-110 may fall under the smallest bf16 (denormals included, which
//    the instruction takes as they are).  What a value leaves after two terms has eight significant
//    bits; they lie in the upper half of the word, where they become the third term, unless that
//    happens.  So: any such remainder with a bit in its lower half, at one operation per pair of values.
//  * The small products of a sum that is itself next to nothing fall under the smallest float32, 2^-149: at most
//    ten cuts of that size, 2^-26 of a result of 2^-119.  So: any accumulator below that, other than zero.
// A tile computed again takes its time and the fp32 instruction's: 4096^3 with every tile 1720 us (700 without, 916 with
// the fp32 instruction alone).  A NaN in one row of A, 32 tiles, takes as long: they run on one XCD, beside workgroups
// whose matrix instructions go first.  Loading the second pass a step ahead changes nothing.
//
// How: a workgroup of four waves owns a BM x BN tile of C (waves 2 x 2), K in steps of 32.  While the
// waves multiply the step in LDS, each thread splits its share of the fp32 values of the next one
// (loaded into registers a step before) and loads the one after it, all in the shadow of the
// matrix instructions; between two barriers the planes of bf16 values then go to LDS.  LDS holds one
// step, 48 KiB for 128 x 128, and two workgroups share a CU: one multiplies while the other writes,
// starts or stores.
//  * Splitting in the copy and not at the operand fetch: every value is split once per workgroup
//    instead of once per wave that reads it.
//  * The differences are plain subtractions: v_dot2c_f32_bf16 would subtract without unpacking, but
//    a matrix instruction next to one takes 36 cycles instead of 16 (measured).
//  * 4096^3 with GELU 916 -> 700 us (196 TFLOP/s of fp32 products, 1180 of bf16 ones), 16 x [256 x 256 x
//    65536] 1015 -> 820, 8192 x 8192 x 32 82 -> 74, 65536 x 128 x 1024 130 -> 101 (fp32 instruction, here).  What bounds
//    it: a step takes 4940 cycles for the pair of workgroups on a CU (3072 are matrix instructions), as
//    splitting, adding and writing take issue slots next to them; the matrix instructions alone, on these
//    operands, run 500 us under the board's power limit.
//  * v_mfma_f32_16x16x32_bf16: with 32x32x16 two LDS stages of 16 k fit, a step takes 3724 cycles per
//    pair of workgroups (3072 are matrix instructions), but the board's power limit then holds the
//    clock at 1.63 GHz (4096^3 in 714 us).
//  * 64 and 32 rows (three workgroups a CU) for outputs of fewer rows: a step of 64 x 128 takes 0.64 of the whole tile's time, of 32 x 128
//    0.48, as the columns are split once for fewer rows (0.88, 0.66 and 1.37 us a step for each workgroup of a full CU, a
//    convolution's input; [16, 448, 704] x [320, 448, 3] 116 us on 128 rows, 80 on 64).
//  * A convolution's input in place (VIEW_INPUT): rows of B are rows of x at an offset, any alignment, so a K step is 32 products whatever
//    the channels and taps, without copies, padding channels or regrouped weights.  Eight lanes follow the wave's eight rows, and a
//    load gets its row by readlane: with the rows in scalar registers of their own the bookkeeping took a third of the issue slots
//    ([11, 256, 24580] x [50, 256, 3] dilation 2: 214 us, 174 so).
// LDS layout: fragments in the order the lanes read them -- sixteen rows x 32 k of one plane are
// one contiguous KiB, lane (k chunk g, row r) reading 16 bytes of 256 g + ... (frag_pos) -- so that
// operand reads need one address register; even rows before odd ones, XORed with the chunk, keeps
// the reads and the writes (every other row, four k chunks at a time) free of bank conflicts.
#ifndef PGK_GEMM_F32_TERMS_H
#define PGK_GEMM_F32_TERMS_H

#include <hip/hip_runtime.h>

#include <cstddef>

#include "pgk_device.h"
#include "pgk_gemm_mfma_kernel.h"
#include "pgk_kernels.h"

namespace pgk {

// f(IC<FROM>{}), ..., f(IC<TO - 1>{}): an unrolled loop whose index is a compile-time constant
template <int FROM, int TO, typename F>
__device__ __forceinline__ void static_for(F&& f)
{
    if constexpr (FROM < TO) {
        f(IC<FROM>{});
        static_for<FROM + 1, TO>(f);
    }
}

// B is the input x of a convolution, x [batch][K / conv_kw][conv_len], read in place: row k of B is the row k / conv_kw of x,
// its element n at n * conv_stride + (k % conv_kw) * conv_dil - conv_pad, zero outside
constexpr int VIEW_INPUT = 2;

template <bool BT_, int BM_, int BN_, int WAVES_PER_SIMD_>
struct TermsCfg {
    static constexpr bool BT = BT_;                    // B given as [N][K]
    static constexpr int BM = BM_, BN = BN_, BK = 32;
    static constexpr int WAVES_PER_SIMD = WAVES_PER_SIMD_;
    static constexpr int WGM = BM >= 64 ? 2 : 1, NW = 4, WGN = NW / WGM, NT = 256;
    static constexpr int WM = BM / WGM, WN = BN / WGN;
    static constexpr int TM16 = WM / 16, TN16 = WN / 16;       // 16 x 16 accumulator blocks per wave
    static constexpr int PLANES = 3;
    static constexpr int BIAS_N = BM > BN ? BM : BN;
    static constexpr int A_PLANE = BM * BK * 2, B_PLANE = BN * BK * 2;     // bytes of one plane
    static constexpr int A_BYTES = PLANES * A_PLANE, B_BYTES = PLANES * B_PLANE;
    // a thread copies two neighbouring rows of A (of a transposed B), columns of a plain B, so many k values of each
    static constexpr int A_KV = BM * BK / NT / 2, B_KV = BN * BK / NT / 2;
    static_assert((A_KV == 8 || A_KV == 4 || A_KV == 2) && B_KV == 8, "pairs of k values; of B a whole chunk");
    // the epilogue stages sixteen rows of a wave's part at a time
    static constexpr int PIECE_BYTES = 16 * WN * 4;
    static_assert(2 * PIECE_BYTES <= A_BYTES && 2 * PIECE_BYTES <= B_BYTES, "epilogue staging");
};

// The epilogue of a wave: its part of the tile, sixteen rows at a time, through a piece of LDS that
// only this wave touches (LDS operations of one wave are carried out in order), stored as whole
// row pieces of WN floats, 16 bytes per lane.  Accumulator layout and KINDs as in
// pgk_gemm_mfma_kernel.h: lane (l16, grp) holds, of block (i, j), row 16 i + l16 and the columns
// 16 j + 4 grp ..; HAS_BIAS false: partial products.
template <int ACT, int KIND, typename Cfg, bool HAS_BIAS, bool STREAM>
__device__ __forceinline__ void epilogue_terms(f32x4 (&acc)[Cfg::TM16][Cfg::TN16], const float* bias, const float* bias_row,
                                               unsigned char* out_tile, size_t ld_bytes, int m_rem, int n_rem, int wm, int wn,
                                               int lane, unsigned char* piece, float* rs_lds)
{
    constexpr int ROWB = Cfg::WN * 4;                     // bytes of a row piece
    constexpr int UNITS = ROWB / 16;
    constexpr int RPP = ROWB >= 256 ? 1 : 256 / ROWB;     // rows per 256-byte bank period
    constexpr int CH = 16 * UNITS / 64;                   // chunks per lane and block
    static_assert(ROWB >= 128 && (16 * UNITS) % 64 == 0, "row pieces of whole lines");
    constexpr bool ROWSUM = KIND == EPI_ROWSUM || KIND == EPI_ROWSUM_MASKED;
    const int grp = lane >> 4, row_in = lane & 15;
    const int wkey = (row_in / RPP) % UNITS;
    // the accumulators of outputs whose row and column are not both odd or both even have their sign turned
    const float sign[2] = {row_in & 1 ? -1.0f : 1.0f, row_in & 1 ? 1.0f : -1.0f};
#pragma unroll
    for (int i = 0; i < Cfg::TM16; ++i) {
        const int row = wm * Cfg::WM + 16 * i + row_in;   // row inside the tile
        float rs = 0.0f, br = 0.0f;
        if constexpr (KIND == EPI_ROWBIAS) br = bias_row[row];
#pragma unroll
        for (int j = 0; j < Cfg::TN16; ++j) {
            const int colw = 16 * j + 4 * grp;            // column inside the wave's part
            const int col = wn * Cfg::WN + colw;
            f32x4 bv = {br, br, br, br};
            if constexpr (HAS_BIAS && KIND != EPI_ROWBIAS) bv = *(const f32x4*)(bias + col);
            int left = n_rem - col;
            // (kept opaque: the comparisons are made where they are used, not held as lane masks)
            if constexpr (KIND == EPI_ROWSUM_MASKED) asm volatile("" : "+v"(left));
            f32x4 y;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if constexpr (HAS_BIAS) y[e] = activate<ACT>(__builtin_fmaf(acc[i][j][e], sign[e & 1], bv[e]));
                else y[e] = __builtin_fmaf(acc[i][j][e], sign[e & 1], 0.0f);
                if constexpr (KIND == EPI_ROWSUM) rs += y[e];
                else if constexpr (KIND == EPI_ROWSUM_MASKED) rs += e < left ? y[e] : 0.0f;
            }
            *(f32x4*)(piece + row_in * ROWB + (((colw >> 2) ^ wkey) * 16)) = y;
        }
        if constexpr (ROWSUM) {
            // the four lanes that share a row, in a fixed order
            rs += __shfl_xor(rs, 16);
            rs += __shfl_xor(rs, 32);
            if (grp == 0) rs_lds[wn * Cfg::BM + row] = rs;
        }
        asm volatile("" ::: "memory");
        u32x4 v[CH];
#pragma unroll
        for (int t = 0; t < CH; ++t) {
            const int c = lane + 64 * t;
            const int r = c / UNITS, cc = c % UNITS;
            v[t] = *(const u32x4*)(piece + r * ROWB + ((cc ^ ((r / RPP) % UNITS)) * 16));
        }
        asm volatile("" ::: "memory");
#pragma unroll
        for (int t = 0; t < CH; ++t) {
            const int c = lane + 64 * t;
            const int r = c / UNITS, cc = c % UNITS;
            const int trow = wm * Cfg::WM + 16 * i + r;
            const int left = n_rem - (wn * Cfg::WN + cc * 4);     // elements of this chunk that exist
            if (trow >= m_rem || left <= 0) continue;
            unsigned char* at = out_tile + (size_t)trow * ld_bytes + (size_t)(wn * Cfg::WN) * 4 + (size_t)cc * 16;
            if (left >= 4) {
                if constexpr (STREAM) __builtin_nontemporal_store(v[t], (u32x4_align4*)at);
                else *(u32x4_align4*)at = v[t];
            } else {
#pragma unroll
                for (int e = 0; e < 3; ++e) {
                    if (e >= left) break;
                    ((unsigned int*)at)[e] = v[t][e];
                }
            }
        }
    }
}

#define PGK_TERMS_LDS(Cfg)                                                                     \
    __shared__ __attribute__((aligned(1024))) unsigned char lds_a[Cfg::A_BYTES];               \
    __shared__ __attribute__((aligned(1024))) unsigned char lds_b[Cfg::B_BYTES];               \
    __shared__ __attribute__((aligned(16))) float rs_buf[Cfg::WGN * Cfg::BM + 2 * Cfg::BIAS_N]

// The tile's statements are text in each kernel and not a function that both call: inlined from one -- whatever it is handed, wherever
// the LDS is declared -- the convolution views' kernel has 18 scalar values too many and keeps them in lanes of vector registers, which every
// tile's start and end pay for ([16, 64, 65536] x [128, 64, 3], six steps a tile: 370 us so, 364 without on the same card).
template <typename Cfg, int VIEW, bool TIMED = false>
__global__ __launch_bounds__(Cfg::NT, Cfg::WAVES_PER_SIMD) void gemm_f32_terms_kernel(const GemmArgs p, const int out_mode)
{
#if defined(__HIP_DEVICE_COMPILE__)
    static_assert(VIEW != VIEW_INPUT, "conv_f32_terms_kernel");
    constexpr bool INSIDE = true;
    PGK_TERMS_LDS(Cfg);
#include "pgk_gemm_f32_terms_tile.h"
#endif
}

template <typename Cfg, int VIEW, bool TIMED, bool INSIDE>
__device__ __forceinline__ void terms_tile(const GemmArgs& p, const int out_mode, unsigned char* const lds_a, unsigned char* const lds_b,
                                           float* const rs_buf)
{
#include "pgk_gemm_f32_terms_tile.h"
}

// A convolution's input read in place
template <typename Cfg>
__global__ __launch_bounds__(Cfg::NT, Cfg::WAVES_PER_SIMD) void conv_f32_terms_kernel(const GemmArgs p)
{
#if defined(__HIP_DEVICE_COMPILE__)
    PGK_TERMS_LDS(Cfg);
    // (the whole tile once for each way: with the branch inside the loop, or a loop for each, registers that cross it are
    // copied and, with 128 rows, spilled)
    const unsigned int tiles = (unsigned int)p.tiles_m * (unsigned int)p.tiles_n;
    int tm, tn;
    tile_coords(xcd_remap(blockIdx.x, gridDim.x) % tiles, p.tiles_m, p.tiles_n, p.group_m, tm, tn);
    const long long from = (long long)tn * Cfg::BN - p.conv_pad;
    const long long to = from + Cfg::BN - 1 + (long long)(p.conv_kw - 1) * p.conv_dil;
    if (p.conv_stride == 1 && from >= 0 && to < p.conv_len && (tn + 1) * Cfg::BN <= p.N)
        terms_tile<Cfg, VIEW_INPUT, false, true>(p, 0, lds_a, lds_b, rs_buf);
    else
        terms_tile<Cfg, VIEW_INPUT, false, false>(p, 0, lds_a, lds_b, rs_buf);
#endif
}

// 128 x 128 tiles: 48 KiB of LDS for operands, two workgroups per CU
using CfgTerms = TermsCfg<false, 128, 128, 2>;
using CfgTermsT = TermsCfg<true, 128, 128, 2>;
// 64 and 32 rows
using CfgTerms64 = TermsCfg<false, 64, 128, 3>;
using CfgTerms32 = TermsCfg<false, 32, 128, 3>;

template <typename Cfg, int VIEW, bool TIMED = false>
static hipError_t launch_terms(const GemmArgs& a, int out_mode, hipStream_t s)
{
    const long long wgs = (long long)a.tiles_m * a.tiles_n * a.batch * a.splits;
    if (wgs <= 0 || wgs > 0x7fffffffLL) return hipErrorInvalidValue;
    if (TIMED != (a.stamps != nullptr)) return hipErrorInvalidValue;
    if constexpr (VIEW == VIEW_INPUT) hipLaunchKernelGGL((conv_f32_terms_kernel<Cfg>), dim3((unsigned int)wgs), dim3(Cfg::NT), 0, s, a);
    else hipLaunchKernelGGL((gemm_f32_terms_kernel<Cfg, VIEW, TIMED>), dim3((unsigned int)wgs), dim3(Cfg::NT), 0, s, a, out_mode);
    return hipGetLastError();
}

}  // namespace pgk
#endif
