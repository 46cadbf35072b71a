// Products of at most 32 rows (a decoding step of a few sequences): C = act(A B + bias), optional row sums.
//
// Such a product is the stream of its one large operand B, read once, and little else.  On 32 x 128 tiles it
// took a K split over workgroups to fill the chip, with partial products in memory, a second launch to
// add them, and copies of operands whose rows start on odd elements.  Here a workgroup owns a few columns
// and all of K: its waves each take a part of K, load both operands straight into
// the registers the matrix instruction reads (no LDS, no barrier on the way; an element's alignment is enough), and add
// their sums through LDS in wave order at the end.  One launch, no workspace (row sums apart).
//
//  * B as [N][K] (a linear layer's weight): four loads of a wave, each of four rows' runs of 256 bytes, become the
//    operands of four instructions by a transposition among neighbouring lanes (transpose_quad).
//  * B as [K][N]: a lane reads VEC neighbouring columns of one k row.  bf16: eight rows, regrouped
//    by v_perm_b32 (one per register read) into VEC fragments of eight k; fp32: the instruction takes one k per
//    lane, so the VEC values are fragments as they are.
//  * bf16 v_mfma_f32_16x16x32_bf16, fp32 v_mfma_f32_16x16x4_f32, columns of B as the first operand: a lane's results
//    are four columns of one row of C.  Rows past M re-read the last one and are not stored.
// Bound by the stream of B and, as it is loaded without LDS, the address path: 8 x 11008 x 4096 bf16, B transposed, 17.5 us
// (5.2 TB/s; 19.7 with tiles, slices and a second pass), fp32 35.2 (41.5).  Tried: non-temporal loads of B (25 us: the two
// halves of a line are read by different instructions), 16 waves or two column blocks per workgroup (no gain), all of a
// wave's steps loaded and then multiplied, batch by batch (plain B 8 x 11008 x 4096 fp32 36 us against 33).
#include <hip/hip_runtime.h>

#include <type_traits>

#include "pgk_device.h"
#include "pgk_kernels.h"

namespace pgk {

namespace {

struct StreamArgs {
    const void* A;       // [batch][M][K]
    const void* B;       // [batch][N][K] or [batch][K][N]
    const float* bias;
    void* C;
    float* rs_part;      // row sums per column group [batch][groups][M] (final with one group), or nullptr
    int M, N, K, act, groups;
};

typedef f32x4 f32x4_align4 __attribute__((aligned(4)));
typedef u32x2 u32x2_align2 __attribute__((aligned(2)));
typedef u32x2 u32x2_align4 __attribute__((aligned(4)));

// The 4 x 4 transposition of 16-byte pieces among four neighbouring lanes: piece t of lane q becomes piece q
// of lane t.  Two exchanges, with the lane beside and the one after that.
__device__ __forceinline__ void transpose_quad(u32x4 (&v)[4], int lane)
{
    const bool odd = lane & 1, high = lane & 2;
    auto beside = [](unsigned int x) { return (unsigned int)__builtin_amdgcn_mov_dpp((int)x, 0xb1, 0xf, 0xf, true); };      // lane ^ 1
    auto across = [](unsigned int x) { return (unsigned int)__builtin_amdgcn_mov_dpp((int)x, 0x4e, 0xf, 0xf, true); };      // lane ^ 2
#pragma unroll
    for (int d = 0; d < 4; ++d) {
#pragma unroll
        for (int t = 0; t < 4; t += 2) {
            const unsigned int x = v[t][d], y = v[t + 1][d], xb = beside(x), yb = beside(y);
            v[t][d] = odd ? yb : x;
            v[t + 1][d] = odd ? y : xb;
        }
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const unsigned int x = v[t][d], y = v[t + 2][d], xb = across(x), yb = across(y);
            v[t][d] = high ? yb : x;
            v[t + 2][d] = high ? y : xb;
        }
    }
}

// BLOCKS: blocks of sixteen columns of a workgroup; for B as [K][N] also the elements a lane loads (VEC)
template <bool BF16, bool BT, int MB, int BLOCKS, int W>
__global__ __launch_bounds__(W * 64) void gemm_stream_kernel(const StreamArgs p)
{
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr int ES = BF16 ? 2 : 4, COLS = 16 * BLOCKS;
    constexpr int KL = BF16 ? 8 : 4;              // k values of sixteen bytes
    // k values of a step.  B transposed: four pieces of a lane, four lane groups; B plain: one piece of each group
    constexpr int KS = BT ? 16 * KL : 4 * KL;
    constexpr int JB = BLOCKS < 2 ? BLOCKS : 2;   // column blocks added up at a time
    __shared__ __attribute__((aligned(16))) f32x4 part[W][MB * JB][64];
    __shared__ __attribute__((aligned(16))) float tile[16 * MB][COLS];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, grp = lane >> 4;
    const int b = blockIdx.x / p.groups, n0 = (blockIdx.x - b * p.groups) * COLS;
    const int M = p.M, N = p.N, K = p.K;
    using elem = typename std::conditional<BF16, unsigned short, float>::type;
    using chunk = typename std::conditional<BF16, u32x4_align2, u32x4_align4>::type;      // sixteen bytes at an element
    const elem* const A = (const elem*)p.A + (size_t)b * (size_t)M * (size_t)K;
    const elem* const B = (const elem*)p.B + (size_t)b * (size_t)N * (size_t)K;

    // B transposed: of sixteen rows of A and of B, load u takes the rows 4 i + u, four neighbouring lanes the four
    // pieces of a lane group's k, so that a load is four runs of 256 bytes; transposed among those lanes, lane
    // (l16, grp) holds the pieces of group grp of row l16, as the instruction takes them.  (Loaded as they are used, a row
    // per lane, the address path takes four times as long: 8 x 11008 x 4096 21.4 us.)  B plain: A as it is used.
    const int k_lane = BT ? KL * (4 * grp + (lane & 3)) : KL * grp, r_lane = BT ? l16 & 12 : l16;
    constexpr int LOADS = BT ? 4 : 1;             // of A per row block and step
    const elem* arow[MB][LOADS];
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int u = 0; u < LOADS; ++u) {
            const int r = 16 * i + r_lane + u;
            arow[i][u] = A + (size_t)(r < M ? r : M - 1) * (size_t)K + k_lane;
        }
    constexpr int VEC = BLOCKS;
    const elem* brow[BT ? BLOCKS : 1][LOADS];
    if constexpr (BT) {
#pragma unroll
        for (int j = 0; j < BLOCKS; ++j)
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int n = n0 + 16 * j + r_lane + u;
                brow[j][u] = B + (size_t)(n < N ? n : N - 1) * (size_t)K + k_lane;
            }
    } else {
        // B plain: this lane's first column (the last VEC columns where its own run past the row's end)
        const int my_col = n0 + VEC * l16 + VEC <= N ? n0 + VEC * l16 : N - VEC;
        brow[0][0] = B + (size_t)k_lane * (size_t)N + my_col;
    }

    f32x4 acc[MB][BLOCKS];
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < BLOCKS; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

    // sixteen bytes of a row (`whole`: the step lies inside K), what lies behind K as zero: a piece that K ends in is
    // read from where it ends with K, and moved (K >= KL)
    auto piece = [&](const elem* row, int step, bool whole) __attribute__((always_inline)) -> u32x4 {
        const elem* const at = row + (size_t)step * KS;
        if (whole) return *(const chunk*)at;
        const int left = K - step * KS - k_lane;           // elements of the piece that exist
        const int back = left >= KL ? 0 : left > 0 ? KL - left : 0;
        const u32x4 v = *(const chunk*)(left > 0 ? at - back : row - k_lane);
        unsigned long long lo = ((unsigned long long)v[1] << 32) | v[0], hi = ((unsigned long long)v[3] << 32) | v[2];
        const unsigned int bits = 8u * ES * (unsigned int)back, sh = bits & 63u;
        const unsigned long long from_hi = sh ? hi << (64u - sh) : 0ull;
        lo = bits >= 64u ? hi >> sh : (lo >> sh) | from_hi;
        hi = bits >= 64u ? 0ull : hi >> sh;
        if (left <= 0) lo = hi = 0ull;
        return u32x4{(unsigned int)lo, (unsigned int)(lo >> 32), (unsigned int)hi, (unsigned int)(hi >> 32)};
    };
    // the products of one piece per row of A, `sa`, with B as loaded, `sb` (BT: a piece per block; else VEC columns of KL rows)
    auto multiply_part = [&](const u32x4 (&sa)[MB], const unsigned int* sb) __attribute__((always_inline)) {
        if constexpr (BF16) {
            bf16x8 fb[BLOCKS];
            if constexpr (BT) {
#pragma unroll
                for (int j = 0; j < BLOCKS; ++j)
                    fb[j] = __builtin_bit_cast(bf16x8, u32x4{sb[4 * j], sb[4 * j + 1], sb[4 * j + 2], sb[4 * j + 3]});
            } else {
                // column j of the lane: the halves j % 2 of register j / 2 of its eight rows, in pairs
#pragma unroll
                for (int j = 0; j < BLOCKS; ++j) {
                    u32x4 f;
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        f[q] = __builtin_amdgcn_perm(sb[(2 * q + 1) * (VEC / 2) + j / 2], sb[2 * q * (VEC / 2) + j / 2],
                                                     j % 2 ? 0x07060302u : 0x05040100u);
                    fb[j] = __builtin_bit_cast(bf16x8, f);
                }
            }
#pragma unroll
            for (int i = 0; i < MB; ++i)
#pragma unroll
                for (int j = 0; j < BLOCKS; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[j], __builtin_bit_cast(bf16x8, sa[i]), acc[i][j], 0, 0, 0);
        } else {
            auto f = [](unsigned int w) __attribute__((always_inline)) { return __builtin_bit_cast(float, w); };
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int i = 0; i < MB; ++i) {
                    const unsigned int aw = sa[i][e];
#pragma unroll
                    for (int j = 0; j < BLOCKS; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(f(BT ? sb[4 * j + e] : sb[e * VEC + j]), f(aw), acc[i][j], 0, 0, 0);
                }
        }
    };

    const int steps = (K + KS - 1) / KS;
    const int s_begin = (int)((long long)wave * steps / W), s_end = (int)((long long)(wave + 1) * steps / W);
    if constexpr (BT) {
        // two steps in flight: one's registers are loaded anew as soon as it is multiplied
        struct Step { u32x4 a[MB][4], b[BLOCKS][4]; };
        Step st[2];
        auto load = [&](Step& s, int step) __attribute__((always_inline)) {
            const bool whole = (step + 1) * KS <= K;
#pragma unroll
            for (int j = 0; j < BLOCKS; ++j)
#pragma unroll
                for (int u = 0; u < 4; ++u) s.b[j][u] = piece(brow[j][u], step, whole);
#pragma unroll
            for (int i = 0; i < MB; ++i)
#pragma unroll
                for (int u = 0; u < 4; ++u) s.a[i][u] = piece(arow[i][u], step, whole);
        };
        auto multiply = [&](Step& s) __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < BLOCKS; ++j) transpose_quad(s.b[j], lane);
#pragma unroll
            for (int i = 0; i < MB; ++i) transpose_quad(s.a[i], lane);
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                u32x4 sa[MB];
                unsigned int sb[4 * BLOCKS];
#pragma unroll
                for (int i = 0; i < MB; ++i) sa[i] = s.a[i][t];
#pragma unroll
                for (int j = 0; j < BLOCKS; ++j)
#pragma unroll
                    for (int d = 0; d < 4; ++d) sb[4 * j + d] = s.b[j][t][d];
                multiply_part(sa, sb);
            }
        };
        if (s_begin < s_end) load(st[0], s_begin);
        if (s_begin + 1 < s_end) load(st[1], s_begin + 1);
        for (int s = s_begin; s < s_end; s += 2) {
            __builtin_amdgcn_sched_barrier(0);
            multiply(st[0]);
            if (s + 2 < s_end) load(st[0], s + 2);
            __builtin_amdgcn_sched_barrier(0);
            if (s + 1 < s_end) {
                multiply(st[1]);
                if (s + 3 < s_end) load(st[1], s + 3);
            }
        }
    } else {
        // DEPTH steps are in flight all the time: a step's registers are loaded anew as soon as it is multiplied
        // (the barriers keep the compiler from gathering the loads behind the arithmetic)
        constexpr int ROW = VEC * ES / 4;         // registers of a lane's row
        constexpr int DEPTH = KL >= 8 ? 2 : 4;
        struct Step { u32x4 a[MB]; unsigned int b[KL * ROW]; };
        Step st[DEPTH];
        auto load_row = [&](const elem* at, unsigned int* to) __attribute__((always_inline)) {       // VEC elements
            if constexpr (VEC * ES == 16) {
                const u32x4 v = *(const chunk*)at;
#pragma unroll
                for (int d = 0; d < 4; ++d) to[d] = v[d];
            } else if constexpr (BF16) {
                const u32x2 v = *(const u32x2_align2*)at;
                to[0] = v[0]; to[1] = v[1];
            } else {
                const u32x2 v = *(const u32x2_align4*)at;
                to[0] = v[0]; to[1] = v[1];
            }
        };
        auto load = [&](Step& s, int step) __attribute__((always_inline)) {
            const elem* const at = brow[0][0] + (size_t)step * KS * (size_t)N;
#pragma unroll
            for (int r = 0; r < KL; ++r) load_row(at + (size_t)r * (size_t)N, s.b + r * ROW);
#pragma unroll
            for (int i = 0; i < MB; ++i) s.a[i] = piece(arow[i][0], step, true);
        };
        const int whole = K / KS, s_whole = s_end < whole ? s_end : whole;
        int s = s_begin;
        if (s + DEPTH <= s_whole) {
#pragma unroll
            for (int u = 0; u < DEPTH; ++u) load(st[u], s + u);
            __builtin_amdgcn_sched_barrier(0);
            for (; s + 2 * DEPTH <= s_whole; s += DEPTH) {
#pragma unroll
                for (int u = 0; u < DEPTH; ++u) {
                    multiply_part(st[u].a, st[u].b);
                    load(st[u], s + DEPTH + u);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            const int more = s_whole - s - DEPTH;         // steps after those in flight, fewer than DEPTH
#pragma unroll
            for (int u = 0; u < DEPTH; ++u) {
                multiply_part(st[u].a, st[u].b);
                if (u < more) load(st[u], s + DEPTH + u);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int u = 0; u < DEPTH - 1; ++u)
                if (u < more) multiply_part(st[u].a, st[u].b);
        } else {
#pragma unroll
            for (int u = 0; u < DEPTH - 1; ++u)
                if (s + u < s_whole) load(st[u], s + u);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < DEPTH - 1; ++u)
                if (s + u < s_whole) multiply_part(st[u].a, st[u].b);
        }
        if (whole >= s_begin && whole < s_end) {          // (the last wave, K not a multiple of the step)
            const int left = K - whole * KS - k_lane;     // rows of this lane that exist
            const elem* const at = brow[0][0] + (size_t)whole * KS * (size_t)N;
#pragma unroll
            for (int r = 0; r < KL; ++r) {
#pragma unroll
                for (int d = 0; d < ROW; ++d) st[0].b[r * ROW + d] = 0u;
                if (r < left) load_row(at + (size_t)r * (size_t)N, st[0].b + r * ROW);
            }
#pragma unroll
            for (int i = 0; i < MB; ++i) st[0].a[i] = piece(arow[i][0], whole, false);
            multiply_part(st[0].a, st[0].b);
        }
    }

    // ---- the waves' sums, added in wave order; the tile of sums in LDS
#pragma unroll
    for (int j0 = 0; j0 < BLOCKS; j0 += JB) {
        if (j0 > 0) __syncthreads();
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
            for (int j = 0; j < JB; ++j) part[wave][i * JB + j][lane] = acc[i][j0 + j];
        __syncthreads();
        for (int t = tid; t < MB * JB * 64; t += W * 64) {
            const int blk = t >> 6, ln = t & 63;
            f32x4 sum = part[0][blk][ln];
#pragma unroll
            for (int w = 1; w < W; ++w) sum += part[w][blk][ln];
            const int row = 16 * (blk / JB) + (ln & 15), j = j0 + blk % JB;
            if constexpr (BT) {
                *(f32x4*)&tile[row][16 * j + 4 * (ln >> 4)] = sum;
            } else {
                // element e is column j of the VEC columns that lane 4 (ln / 16) + e has loaded; where those
                // were moved back from the row's end, the ones that are another lane's are left to that one
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int c = VEC * (4 * (ln >> 4) + e), at = n0 + c + VEC <= N ? c : N - VEC - n0;
                    if (at + j >= c) tile[row][at + j] = sum[e];
                }
            }
        }
    }
    __syncthreads();

    // ---- bias, activation, store, row sums: four columns per thread
    constexpr int G = COLS / 4;
    for (int t = tid; t < 16 * MB * G; t += W * 64) {
        const int row = t / G, col = 4 * (t % G), n = n0 + col;
        const int left = N - n;                     // columns that exist
        float y[4], rs = 0.0f;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float add = p.bias && e < left ? p.bias[n + e] : 0.0f;
            y[e] = e < left ? activate_dyn(tile[row][col + e] + add, p.act) : 0.0f;
            rs += y[e];
        }
        if (row < M && left > 0) {
            elem* const c = (elem*)p.C + ((size_t)b * (size_t)M + row) * (size_t)N + n;
            if constexpr (BF16) {
                const unsigned int lo = pack_bf16x2(y[0], y[1]), hi = pack_bf16x2(y[2], y[3]);
                if (left >= 4) {
                    *(u32x2_align2*)c = u32x2{lo, hi};
                } else {
                    c[0] = (unsigned short)(lo & 0xffffu);
                    if (left > 1) c[1] = (unsigned short)(lo >> 16);
                    if (left > 2) c[2] = (unsigned short)(hi & 0xffffu);
                }
            } else {
                if (left >= 4) {
                    *(f32x4_align4*)c = f32x4{y[0], y[1], y[2], y[3]};
                } else {
                    c[0] = y[0];
                    if (left > 1) c[1] = y[1];
                    if (left > 2) c[2] = y[2];
                }
            }
        }
        if (p.rs_part) {
            // the G threads of a row are neighbouring lanes: a fixed butterfly
#pragma unroll
            for (int off = 1; off < G; off <<= 1) rs += __shfl_xor(rs, off);
            if (t % G == 0 && row < M) p.rs_part[((size_t)b * p.groups + n0 / COLS) * (size_t)M + row] = rs;
        }
    }
#endif
}

// rowsum[b][m]: the column groups' partial sums, a wave per output (a thread alone, as in
// rowsum_combine_kernel, would wait for hundreds of loads one batch after the other)
__global__ __launch_bounds__(256) void stream_rowsum_kernel(const float* __restrict__ part, float* __restrict__ rowsum, int M,
                                                            long long total, int groups)
{
    const long long i = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (i >= total) return;
    const int lane = threadIdx.x & 63;
    const long long b = i / M, m = i - b * M;
    const float* src = part + b * (long long)groups * M + m;
    float s = 0.0f;
    for (int g = lane; g < groups; g += 64) s += src[(long long)g * M];
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off);
    if (lane == 0) rowsum[i] = s;
}

// (what stream_plan asks for: eight waves but with two blocks; sixteen, bf16 beyond a K of 8192, for which eight blocks would not
// have the registers; four, a plain B up to a K of 1024)
template <bool BF16, bool BT, int MB, int BLOCKS>
hipError_t launch_waves(const StreamArgs& a, int waves, unsigned int wgs, hipStream_t s)
{
    if constexpr (BLOCKS != 2)
        if (waves == 8) {
            hipLaunchKernelGGL((gemm_stream_kernel<BF16, BT, MB, BLOCKS, 8>), dim3(wgs), dim3(512), 0, s, a);
            return hipGetLastError();
        }
    if constexpr (BF16 && BLOCKS < 8)
        if (waves == 16) {
            hipLaunchKernelGGL((gemm_stream_kernel<BF16, BT, MB, BLOCKS, 16>), dim3(wgs), dim3(1024), 0, s, a);
            return hipGetLastError();
        }
    if constexpr (!BT)
        if (waves == 4) {
            hipLaunchKernelGGL((gemm_stream_kernel<BF16, BT, MB, BLOCKS, 4>), dim3(wgs), dim3(256), 0, s, a);
            return hipGetLastError();
        }
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_gemm_stream(const StreamPlan& pl, const void* A, const void* B, const float* bias, void* C, float* rowsum,
                              float* part, int M, int N, int K, int batch, int act, int dtype, bool b_trans, hipStream_t s)
{
    const long long wgs = (long long)pl.groups * batch;
    if (M < 1 || M > 32 || wgs <= 0 || !stream_launch_fits(pl, batch) || N < (b_trans ? 1 : pl.blocks) || K < 8) return hipErrorInvalidValue;
    if ((long long)pl.groups * 16 * pl.blocks < N) return hipErrorInvalidValue;
    const StreamArgs a{A, B, bias, C, !rowsum ? nullptr : pl.groups == 1 ? rowsum : part, M, N, K, act, pl.groups};
    const unsigned int g = (unsigned int)wgs;
    hipError_t e = hipErrorInvalidValue;
    const bool few = M <= 16;
    if (b_trans) {
        if (pl.blocks == 1 && few)
            e = dtype == DT_BF16 ? launch_waves<true, true, 1, 1>(a, pl.waves, g, s) : launch_waves<false, true, 1, 1>(a, pl.waves, g, s);
    } else if (dtype == DT_BF16) {
        if (pl.blocks == 4) e = few ? launch_waves<true, false, 1, 4>(a, pl.waves, g, s) : launch_waves<true, false, 2, 4>(a, pl.waves, g, s);
        if (pl.blocks == 8) e = few ? launch_waves<true, false, 1, 8>(a, pl.waves, g, s) : launch_waves<true, false, 2, 8>(a, pl.waves, g, s);
    } else if (few) {
        if (pl.blocks == 2) e = launch_waves<false, false, 1, 2>(a, pl.waves, g, s);
        if (pl.blocks == 4) e = launch_waves<false, false, 1, 4>(a, pl.waves, g, s);
    }
    if (e != hipSuccess || !rowsum || pl.groups == 1) return e;
    const long long total = (long long)M * batch;
    hipLaunchKernelGGL(stream_rowsum_kernel, dim3((unsigned int)((total + 3) / 4)), dim3(256), 0, s, part, rowsum, M, total, pl.groups);
    return hipGetLastError();
}

}  // namespace pgk
