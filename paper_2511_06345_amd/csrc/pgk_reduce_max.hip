// Maximum over one dimension of a contiguous tensor viewed as [outer][red][inner]:
//     out[o][i] = max_r X[o][r][i],   idx[o][i] = smallest r attaining it
// (the reduction operator of PRAGMA's GPU case study, Section 4.4; the paper gives no
// formula, so this is the plain definition).  IEEE comparison: +0 and -0 tie and the
// earlier one is returned; a NaN in the slice gives that NaN and the first NaN's position.
//
// The kernels are streaming kernels bound by HBM bandwidth: every element is read once, with 16-byte loads
// and several of them in flight per lane.  Where rows do not start on 16-byte boundaries, long ones are
// read in aligned chunks with the elements at their ends apart, shorter and strided ones in chunks from any element on,
// and small problems one element per load (plan_reduce_max).
//   * inner == 1 (the reduced dimension is contiguous): some lanes of a wave (short rows), a wave or a workgroup hold a row in
//     registers, in 16-byte chunks all loaded at once; longer ones are swept by a workgroup.  The maximum comes first, its position after.
//   * 1 < inner, up to about half of what a workgroup loads at once, blocks large enough (plan_block): a workgroup sweeps its block of whole r as it
//     lies in memory, 16 bytes per lane, and combines the lanes of equal inner position through LDS.
//   * inner beyond that, and smaller blocks: lanes lie along the contiguous inner dimension, 16 bytes each; the four
//     waves of a workgroup take every fourth r and are combined through LDS.
// Every combination step compares (value, position) pairs, so the result does not depend
// on how the work was split.  When there are too few outputs to fill the chip the reduced
// range is cut into segments (one workgroup each) and a second small kernel combines the
// segment results in order.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "pgk_device.h"
#include "pgk_kernels.h"

namespace pgk {

namespace {

constexpr float kNegInf = -__builtin_huge_valf();
constexpr int kNoPos = 0x7fffffff;      // position of "no element seen"

// Does (xv at position xi) win over (mv at position mi)?  Positions differ unless both
// are kNoPos.  First NaN wins over everything; otherwise the larger value, and among
// equal values the earlier position.
__device__ __forceinline__ bool beats(float xv, int xi, float mv, int mi)
{
    const bool xn = xv != xv, mn = mv != mv;
    if (xn | mn) return xn && (!mn || xi < mi);
    return xv > mv || (xv == mv && xi < mi);
}

// The same for a scan in increasing position (xi > mi always): x replaces m when it is
// larger or the first NaN; an equal x never does.
__device__ __forceinline__ bool replaces(float xv, float mv) { return !(xv <= mv) && mv == mv; }

template <bool BF16>
struct Elem {
    static constexpr int BYTES = BF16 ? 2 : 4;
    static constexpr int VEC = 16 / BYTES;          // elements per 16-byte chunk
};

// widen the VEC elements of one 16-byte chunk to float (exact)
template <bool BF16>
__device__ __forceinline__ void unpack(const u32x4& w, float (&x)[Elem<BF16>::VEC])
{
    if constexpr (BF16) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const unsigned int lo = w[q] << 16, hi = w[q] & 0xffff0000u;
            x[2 * q] = __builtin_bit_cast(float, lo);
            x[2 * q + 1] = __builtin_bit_cast(float, hi);
        }
    } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const unsigned int bits = w[q];       // a value, not a vector-element lvalue, for the bit cast
            x[q] = __builtin_bit_cast(float, bits);
        }
    }
}

// one 16-byte chunk, aligned or (UNALIGNED) starting on any element
template <bool BF16, bool UNALIGNED>
__device__ __forceinline__ u32x4 load_chunk(const unsigned char* at)
{
    using any_element = typename std::conditional<BF16, u32x4_align2, u32x4_align4>::type;
    if constexpr (UNALIGNED) return __builtin_nontemporal_load((const any_element*)at);
    else return __builtin_nontemporal_load((const u32x4*)at);
}

template <bool BF16>
__device__ __forceinline__ float load_one(const void* X, size_t e)
{
    if constexpr (BF16) return __builtin_bit_cast(float, (unsigned int)((const unsigned short*)X)[e] << 16);
    else return ((const float*)X)[e];
}

template <bool BF16>
__device__ __forceinline__ void store_one(void* out, size_t e, float v)
{
    if constexpr (BF16) ((unsigned short*)out)[e] = (unsigned short)(__builtin_bit_cast(unsigned int, v) >> 16);
    else ((float*)out)[e] = v;
}

// ---------------------------------------------------------------------------------
// Rows (inner == 1): the largest value first, then where it is.  A compare, a select of the value and one of its position per element
// are four to six operations, and bound rows by the vector ALU: bf16 ones of 520 elements streamed at 3.3 TB/s, of 100 at 1.1.
// v_maximum3_f32 takes two elements at a time and hands NaN on, and the position is looked up once, in what the maximum came
// from: both stream at 5.3 to 7.0.  (Its maximum orders -0 below +0: what is looked up is the first element that compares equal.)
__device__ __forceinline__ float maximum(float a, float b) { return __builtin_elementwise_maximum(a, b); }

template <bool BF16>
__device__ __forceinline__ float chunk_maximum(const u32x4& w)
{
    constexpr int VEC = Elem<BF16>::VEC;
    float x[VEC];
    unpack<BF16>(w, x);
    float m = x[0];
#pragma unroll
    for (int e = 1; e < VEC; ++e) m = maximum(m, x[e]);
    return m;
}
template <bool BF16>
__device__ __forceinline__ float chunk_maximum(float x) { return x; }

// Is x what the maximum m stands for?  NANS: where m may be one.
template <bool NANS>
__device__ __forceinline__ bool is_maximum(float x, float m) { return NANS ? x == m || (x != x && m != m) : x == m; }

// Of U chunks in ascending position with their maxima, the first element that m stands for: its value, its chunk and its place there
// (false: none).
template <bool BF16, bool NANS, int U>
__device__ __forceinline__ bool first_of(const u32x4 (&w)[U], const float (&cm)[U], float m, float& v, int& chunk, int& e0)
{
    constexpr int VEC = Elem<BF16>::VEC;
    u32x4 sel = w[U - 1];
    chunk = U - 1;
#pragma unroll
    for (int u = U - 2; u >= 0; --u)
        if (is_maximum<NANS>(cm[u], m)) { sel = w[u]; chunk = u; }
    float x[VEC];
    unpack<BF16>(sel, x);
    e0 = -1;
    v = 0.0f;
#pragma unroll
    for (int e = VEC - 1; e >= 0; --e)
        if (is_maximum<NANS>(x[e], m)) { e0 = e; v = x[e]; }
    return e0 >= 0;
}
template <bool BF16, bool NANS, int U>
__device__ __forceinline__ bool first_of(const float (&w)[U], const float (&cm)[U], float m, float& v, int& chunk, int& e0)
{
    chunk = -1;
    v = 0.0f;
    e0 = 0;
#pragma unroll
    for (int u = U - 1; u >= 0; --u)
        if (is_maximum<NANS>(cm[u], m)) { v = w[u]; chunk = u; }
    return chunk >= 0;
}

// `combine` over the 1 << lg lanes of a group, in every one of them
template <typename T, typename F>
__device__ __forceinline__ T across(T v, int lg, F combine)
{
    auto dpp = [&](auto ctrl) { return __builtin_bit_cast(T, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), decltype(ctrl)::value, 0xf, 0xf, true)); };
    if (lg >= 1) v = combine(v, dpp(std::integral_constant<int, 0xB1>{}));       // quad_perm [1, 0, 3, 2]
    if (lg >= 2) v = combine(v, dpp(std::integral_constant<int, 0x4E>{}));       // quad_perm [2, 3, 0, 1]
    if (lg >= 3) v = combine(v, dpp(std::integral_constant<int, 0x141>{}));      // row_half_mirror
    if (lg >= 4) v = combine(v, dpp(std::integral_constant<int, 0x140>{}));      // row_mirror
    if (lg >= 5) {
        const auto s = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned int, v), __builtin_bit_cast(unsigned int, v), false, false);
        const unsigned int s0 = s[0], s1 = s[1];
        v = combine(__builtin_bit_cast(T, s0), __builtin_bit_cast(T, s1));
    }
    if (lg >= 6) {
        const auto s = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned int, v), __builtin_bit_cast(unsigned int, v), false, false);
        const unsigned int s0 = s[0], s1 = s[1];
        v = combine(__builtin_bit_cast(T, s0), __builtin_bit_cast(T, s1));
    }
    return v;
}
__device__ __forceinline__ float across_max(float v, int lg) { return across(v, lg, [](float a, float b) { return maximum(a, b); }); }
__device__ __forceinline__ int across_min(int v, int lg) { return across(v, lg, [](int a, int b) { return a < b ? a : b; }); }

// Rows held in registers: g = 1 << lg lanes of a wave (G == 64), or the workgroup (256, 512 or 1024 threads), share a row, U chunks of 16 bytes
// per lane, all loaded at once.  ANY: rows start on any element.  Either way a chunk that would reach past the row's end is moved back to end with it: the
// elements it shares with others are found at the same positions.  LEAD: aligned chunks, the last one in place of those past it, the elements at the
// row's ends apart, one per lane (bf16 rows of 9999 elements: 56 us with ANY, 44 so; in a wave's lanes ANY is faster, of 333: 48 and 60; fp32 alike).
// VEC == 1: rows shorter than a chunk, one lane each.
enum { ALIGNED, ANY, LEAD };

template <bool BF16, int VEC, int FORM, int U, int G>
__global__ __launch_bounds__(G > 64 ? G : 256) void reduce_max_held_rows_kernel(const void* __restrict__ X, void* __restrict__ out,
                                                                   int* __restrict__ idx, long long outer, int red, int lg)
{
    __shared__ float sv[G > 64 ? G / 64 : 1];
    __shared__ int si[G > 64 ? G / 64 : 1];
    const int tid = threadIdx.x;
    const int g = G > 64 ? G : 1 << lg;
    const int gl = tid & (g - 1);
    const long long row = G > 64 ? (long long)blockIdx.x : (long long)blockIdx.x * (256 >> lg) + (tid >> lg);
    const bool active = row < outer;              // whole groups only
    const size_t row_base = (size_t)(active ? row : outer - 1) * (size_t)red;
    const unsigned char* const row_at = (const unsigned char*)X + row_base * Elem<BF16>::BYTES;
    const int lead = FORM == LEAD ? (int)((0u - (unsigned int)(size_t)row_at) & 15u) / Elem<BF16>::BYTES : 0;
    const int nch = (red - lead) / VEC, rest = red - lead - nch * VEC;      // (with LEAD)
    auto start = [&](int c) __attribute__((always_inline)) {
        if constexpr (FORM == LEAD) return lead + (c < nch ? c : nch - 1) * VEC;
        else return c * VEC < red - VEC ? c * VEC : red - VEC;
    };
    using loaded = typename std::conditional<VEC == 1, float, u32x4>::type;
    loaded w[U];
    float cm[U];
    float lead_v = kNegInf, rest_v = kNegInf;
    if constexpr (FORM == LEAD) {
        if (gl < lead) lead_v = load_one<BF16>(X, row_base + gl);
        if (gl < rest) rest_v = load_one<BF16>(X, row_base + red - rest + gl);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        if constexpr (VEC == 1) w[u] = load_one<BF16>(X, row_base + start(gl + u * g));
        else w[u] = load_chunk<BF16, FORM == ANY>(row_at + (size_t)start(gl + u * g) * Elem<BF16>::BYTES);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) cm[u] = chunk_maximum<BF16>(w[u]);
    float m = cm[0];
#pragma unroll
    for (int u = 1; u < U; ++u) m = maximum(m, cm[u]);
    if constexpr (FORM == LEAD) m = maximum(m, maximum(lead_v, rest_v));
    const int wave_lg = G > 64 ? 6 : lg;
    m = across_max(m, wave_lg);
    float v;
    int chunk, e;
    bool found;
    if (__any(m != m)) found = first_of<BF16, true, U>(w, cm, m, v, chunk, e);
    else found = first_of<BF16, false, U>(w, cm, m, v, chunk, e);
    int pos = found ? start(gl + chunk * g) + e : kNoPos;
    if constexpr (FORM == LEAD) {
        if (!found && gl < rest && is_maximum<true>(rest_v, m)) { v = rest_v; pos = red - rest + gl; }
        if (gl < lead && is_maximum<true>(lead_v, m)) { v = lead_v; pos = gl; }
    }
    const int first = across_min(pos, wave_lg);
    if constexpr (G > 64) {
        if (pos == first) { sv[tid >> 6] = v; si[tid >> 6] = pos; }      // (lanes that share an element write the same)
        __syncthreads();
        if (tid == 0) {
            v = sv[0];
            pos = si[0];
#pragma unroll
            for (int q = 1; q < G / 64; ++q)
                if (beats(sv[q], si[q], v, pos)) { v = sv[q]; pos = si[q]; }
            store_one<BF16>(out, (size_t)row, v);
            if (idx) idx[row] = pos;
        }
    } else if (active && pos == first) {
        store_one<BF16>(out, (size_t)row, v);
        if (idx) idx[row] = pos;
    }
}

// Longer rows: the workgroup sweeps the chunks [c0, c1) of one row, UNROLL sweeps at a time (the last chunk in place of those past
// it); a lane keeps its maximum and the sweeps it came from, and the first of those that have the row's read theirs again for the position.
// ENDS: the rows do not all start on 16-byte boundaries; the elements before a row's first boundary and those behind its last
// whole chunk are taken one per lane (bf16 [2048, 50257]: 105 us with one element per load, 39 so).
// Result: direct to out / idx when segs == 1, else to the segment partials.
template <bool BF16, bool ENDS, int UNROLL>
__global__ __launch_bounds__(256) void reduce_max_rows_kernel(const void* __restrict__ X, void* __restrict__ out,
                                                              int* __restrict__ idx, float* __restrict__ pv,
                                                              int* __restrict__ pi, int red, int segs, int chunks_per_seg)
{
    constexpr int VEC = Elem<BF16>::VEC, G = 256;
    __shared__ float sv[4];
    __shared__ int si[4];
    const int gl = threadIdx.x;
    const long long unit = blockIdx.x;            // row * segs + seg
    const long long row = unit / segs;
    const int seg = (int)(unit - row * segs);
    const size_t row_base = (size_t)row * (size_t)red;
    const unsigned char* const row_at = (const unsigned char*)X + row_base * Elem<BF16>::BYTES;
    // elements before the first 16-byte boundary (red is larger than that), whole chunks, elements left
    const int lead = ENDS ? (int)((0u - (unsigned int)(size_t)row_at) & 15u) / Elem<BF16>::BYTES : 0;
    const int nch = (red - lead) / VEC;
    const int rest = ENDS ? red - lead - nch * VEC : 0;
    const int c0 = seg * chunks_per_seg;
    const int c1 = c0 + chunks_per_seg < nch ? c0 + chunks_per_seg : nch;
    const u32x4* const src = (const u32x4*)(row_at + lead * Elem<BF16>::BYTES);

    // (the elements at the row's ends: the first segment's lanes and the last one's)
    float lead_v = kNegInf, rest_v = kNegInf;
    const bool has_lead = ENDS && seg == 0 && gl < lead, has_rest = ENDS && seg == segs - 1 && gl < rest;
    if constexpr (ENDS) {
        if (has_lead) lead_v = load_one<BF16>(X, row_base + gl);
        if (has_rest) rest_v = load_one<BF16>(X, row_base + red - rest + gl);
    }
    // chunks first + gl, first + gl + G, ... (past the end: the last one)
    auto load = [&](int first, u32x4 (&w)[UNROLL]) __attribute__((always_inline)) {
        const int at = first < c1 ? first : c1 - 1, left = c1 - 1 - at;
        const unsigned char* const from = (const unsigned char*)(src + at);
        const unsigned int most = 16u * (unsigned int)(left < UNROLL * G ? left : UNROLL * G);
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            const unsigned int off = 16u * (unsigned int)(gl + u * G);
            w[u] = __builtin_nontemporal_load((const u32x4*)(from + (off < most ? off : most)));
        }
    };
    float best = kNegInf;
    int best_first = c0;                          // the sweeps it came from
    auto take = [&](int first, const u32x4 (&w)[UNROLL]) __attribute__((always_inline)) {
        float m = chunk_maximum<BF16>(w[0]);
#pragma unroll
        for (int u = 1; u < UNROLL; ++u) m = maximum(m, chunk_maximum<BF16>(w[u]));
        if (replaces(m, best)) { best = m; best_first = first; }
    };
    if (c0 < c1) {                                // (as many sweeps are on their way as are looked at)
        u32x4 w0[UNROLL], w1[UNROLL];
        load(c0, w0);
        for (int c = c0; c < c1; c += 2 * UNROLL * G) {
            load(c + UNROLL * G, w1);
            take(c, w0);
            if (c + UNROLL * G >= c1) break;
            load(c + 2 * UNROLL * G, w0);
            take(c + UNROLL * G, w1);
        }
    }
    float m = maximum(maximum(lead_v, rest_v), best);
    m = across_max(m, 6);
    int pos = kNoPos;
    float v = m;
    const bool has = c0 < c1 && is_maximum<true>(best, m);
    // (of the wave's lanes that have it those of the earliest sweeps: bf16 values tie often)
    const int earliest = across_min(has ? best_first : kNoPos, 6);
    if (has && best_first == earliest) {
        u32x4 w[UNROLL];
        float cm[UNROLL];
        load(best_first, w);
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) cm[u] = chunk_maximum<BF16>(w[u]);
        int chunk, e;
        float x;
        if (first_of<BF16, true, UNROLL>(w, cm, m, x, chunk, e)) {
            const int c = best_first + gl + chunk * G;
            v = x;
            pos = lead + (c < c1 ? c : c1 - 1) * VEC + e;
        }
    }
    if constexpr (ENDS) {
        if (has_rest && pos == kNoPos && is_maximum<true>(rest_v, m)) { v = rest_v; pos = red - rest + gl; }
        if (has_lead && is_maximum<true>(lead_v, m)) { v = lead_v; pos = gl; }
    }
    const int first = across_min(pos, 6);
    if (pos == first) { sv[gl >> 6] = v; si[gl >> 6] = pos; }            // (lanes that share an element write the same)
    __syncthreads();
    if (gl != 0) return;
    v = sv[0];
    pos = si[0];
#pragma unroll
    for (int q = 1; q < 4; ++q)
        if (beats(sv[q], si[q], v, pos)) { v = sv[q]; pos = si[q]; }
    if (segs == 1) {
        store_one<BF16>(out, (size_t)row, v);
        if (idx) idx[row] = pos;
    } else {
        pv[unit] = v;
        pi[unit] = pos;
    }
}

// ---------------------------------------------------------------------------------
// inner > 1.  A workgroup owns 64 * VEC consecutive inner positions of one outer index
// and the r range of one segment; wave w takes r = r0 + w, r0 + w + 4, ...  UNALIGNED: rows of inner
// elements that do not all start on 16-byte boundaries are read in 16-byte chunks all the same, from
// any element on (fp32 [215, 6701, 135]: 752 us with one element per load, 139 so); the last lane's chunk
// ends with the row (and overlaps the one before: the outputs
// they share are written twice, with the same values).  VEC == 1: one element per load, for the unaligned
// problems that plan_reduce_max gives to it.
template <bool BF16, int VEC, bool UNALIGNED>
__global__ __launch_bounds__(256) void reduce_max_cols_kernel(const void* __restrict__ X, void* __restrict__ out,
                                                              int* __restrict__ idx, float* __restrict__ pv,
                                                              int* __restrict__ pi, long long outer, int red,
                                                              long long inner, int tiles_i, int segs, int r_per_seg)
{
    // loads in flight per lane: four for fp32; two for bf16, whose eight slots per load keep the
    // vector ALU busier (measured on [32, 4096, 4096] bf16: 6000 GB/s with two, 5700 with four, 5350 with eight)
    constexpr int UNROLL = BF16 && VEC > 1 ? 2 : 4;
    __shared__ float sv[3][64 * VEC];
    __shared__ int si[3][64 * VEC];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    long long u = blockIdx.x;
    const int ti = (int)(u % tiles_i); u /= tiles_i;
    const int seg = (int)(u % segs);
    const long long o = u / segs;
    const long long i_lane = (long long)ti * (64 * VEC) + (long long)lane * VEC;
    const bool in_range = i_lane < inner;         // (aligned rows: inner is a multiple of VEC)
    const long long i0 = UNALIGNED && i_lane + VEC > inner ? inner - VEC : i_lane;
    const int r0 = seg * r_per_seg;
    const int r1 = r0 + r_per_seg < red ? r0 + r_per_seg : red;

    float bv[VEC];
    int bp[VEC];
#pragma unroll
    for (int e = 0; e < VEC; ++e) { bv[e] = kNegInf; bp[e] = kNoPos; }

    if (in_range) {
        const size_t base = ((size_t)o * (size_t)red) * (size_t)inner + (size_t)i0;   // element index of r = 0
        int r = r0 + wave;
        // the wave's first element starts the scan (so the loops need no "nothing seen yet" test)
        const unsigned char* src = (const unsigned char*)X + base * Elem<BF16>::BYTES;
        const size_t rstride = (size_t)inner * Elem<BF16>::BYTES;
        using loaded = typename std::conditional<VEC == 1, float, u32x4>::type;
        auto load = [&](int at) -> loaded {
            if constexpr (VEC == 1) return load_one<BF16>(X, base + (size_t)at * (size_t)inner);
            else return load_chunk<BF16, UNALIGNED>(src + (size_t)at * rstride);
        };
        auto values = [](const loaded& w, float (&x)[VEC]) {
            if constexpr (VEC == 1) x[0] = w;
            else unpack<BF16>(w, x);
        };
        if (r < r1) {
            values(load(r), bv);
#pragma unroll
            for (int e = 0; e < VEC; ++e) bp[e] = r;
            r += 4;
        }
        for (; r + (UNROLL - 1) * 4 < r1; r += UNROLL * 4) {
            loaded w[UNROLL];
#pragma unroll
            for (int q = 0; q < UNROLL; ++q) w[q] = load(r + 4 * q);
#pragma unroll
            for (int q = 0; q < UNROLL; ++q) {
                float x[VEC];
                values(w[q], x);
#pragma unroll
                for (int e = 0; e < VEC; ++e)
                    if (replaces(x[e], bv[e])) { bv[e] = x[e]; bp[e] = r + 4 * q; }
            }
        }
        for (; r < r1; r += 4) {
            float x[VEC];
            values(load(r), x);
#pragma unroll
            for (int e = 0; e < VEC; ++e)
                if (replaces(x[e], bv[e])) { bv[e] = x[e]; bp[e] = r; }
        }
    }
    // waves 1..3 hand their results to wave 0
    if (wave > 0) {
#pragma unroll
        for (int e = 0; e < VEC; ++e) { sv[wave - 1][lane * VEC + e] = bv[e]; si[wave - 1][lane * VEC + e] = bp[e]; }
    }
    __syncthreads();
    if (wave == 0 && in_range) {
#pragma unroll
        for (int w = 0; w < 3; ++w)
#pragma unroll
            for (int e = 0; e < VEC; ++e) {
                const float ov = sv[w][lane * VEC + e];
                const int op = si[w][lane * VEC + e];
                if (beats(ov, op, bv[e], bp[e])) { bv[e] = ov; bp[e] = op; }
            }
        const size_t dst = (size_t)o * (size_t)inner + (size_t)i0;
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            if (segs == 1) {
                store_one<BF16>(out, dst + e, bv[e]);
                if (idx) idx[dst + e] = bp[e];
            } else {
                const size_t at = ((size_t)o * segs + seg) * (size_t)inner + (size_t)i0 + e;
                pv[at] = bv[e];
                pi[at] = bp[e];
            }
        }
    }
}

// ---------------------------------------------------------------------------------
// 1 < inner <= 64 (the blocks that plan_block does not give to the kernel after this one).  One wave owns one outer index (and the r range of one segment) and sweeps that contiguous
// block of red x inner elements: R = 64 / inner consecutive r at a time, lane l at inner
// position l % inner of r number l / inner of the sweep -- 64 (or R * inner) consecutive
// elements per load instruction, eight sweeps in flight.  The lanes that share an inner
// position are then combined through LDS.
template <bool BF16>
__global__ __launch_bounds__(256) void reduce_max_small_inner_kernel(const void* __restrict__ X, void* __restrict__ out,
                                                                     int* __restrict__ idx, float* __restrict__ pv,
                                                                     int* __restrict__ pi, long long outer, int red,
                                                                     int inner, int segs, int r_per_seg)
{
    constexpr int UNROLL = 8;
    __shared__ float sv[4][64];
    __shared__ int si[4][64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const long long unit = (long long)blockIdx.x * 4 + wave;        // o * segs + seg
    const bool active = unit < outer * segs;                        // uniform per wave
    const long long o = active ? unit / segs : 0;
    const int seg = active ? (int)(unit - o * segs) : 0;
    const int R = 64 / inner, L = R * inner;
    const int i = lane % inner, rr = lane / inner;
    const bool lane_ok = active && lane < L;
    const int r0 = seg * r_per_seg;
    const int r1 = active ? (r0 + r_per_seg < red ? r0 + r_per_seg : red) : r0;
    const size_t base = (size_t)o * (size_t)red * (size_t)inner + (size_t)i;

    float bv = kNegInf;
    int bp = kNoPos;
    int r = r0 + rr;
    if (lane_ok && r < r1) { bv = load_one<BF16>(X, base + (size_t)r * inner); bp = r; }   // starts the scan
    r += R;
    for (; r - rr + (UNROLL - 1) * R < r1; r += UNROLL * R) {       // uniform: all UNROLL sweeps start inside the range
        float x[UNROLL];
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            const int ru = r + u * R;
            x[u] = (lane_ok && ru < r1) ? load_one<BF16>(X, base + (size_t)ru * inner) : kNegInf;
        }
#pragma unroll
        for (int u = 0; u < UNROLL; ++u)
            if (lane_ok && r + u * R < r1 && replaces(x[u], bv)) { bv = x[u]; bp = r + u * R; }
    }
    for (; r - rr < r1; r += R) {
        if (lane_ok && r < r1) {
            const float x = load_one<BF16>(X, base + (size_t)r * inner);
            if (replaces(x, bv)) { bv = x; bp = r; }
        }
    }
    sv[wave][lane] = bv;
    si[wave][lane] = bp;
    __syncthreads();
    if (active && lane < inner) {
        float v = sv[wave][lane];
        int p = si[wave][lane];
        for (int q = 1; q < R; ++q) {
            const float ov = sv[wave][q * inner + lane];
            const int op = si[wave][q * inner + lane];
            if (beats(ov, op, v, p)) { v = ov; p = op; }
        }
        if (segs == 1) {
            store_one<BF16>(out, (size_t)o * inner + lane, v);
            if (idx) idx[(size_t)o * inner + lane] = p;
        } else {
            const size_t at = ((size_t)o * segs + seg) * (size_t)inner + lane;
            pv[at] = v;
            pi[at] = p;
        }
    }
}

// ---------------------------------------------------------------------------------
// inner up to about half the elements a workgroup loads at once.  A workgroup owns one outer index (and the r range of one
// segment), a contiguous block of elements, and sweeps it in periods of R x inner of them, R whole r: 16 bytes per
// lane, all lanes side by side whatever inner is, UNROLL periods in flight.  What a lane's element e of every period has in
// common is its inner position, so it keeps the best (value, period) of it; the R entries that share an inner position
// are combined at the end through LDS, a quarter of the rows left at a time.  A period that is a multiple of the
// chunk starts on 16-byte boundaries wherever X starts (`lead` elements before the block); others are read from
// any element on.
// Bound by memory: bf16 [220, 50560, 7] 35 us (112 with a wave per segment and one element per load, which the address path
// bounds), [128, 24742, 88] 90 (322 in the strided kernel, of whose lanes inner / (64 VEC) are at work: 6.3 TB/s), fp32 [200, 20000, 40] 105 (260).
template <bool BF16, int NT>
__global__ __launch_bounds__(NT) void reduce_max_block_kernel(const void* __restrict__ X, void* __restrict__ out,
                                                              int* __restrict__ idx, float* __restrict__ pv,
                                                              int* __restrict__ pi, int red, int inner, int segs,
                                                              int r_per_seg, int R)
{
    constexpr int VEC = Elem<BF16>::VEC, ES = Elem<BF16>::BYTES, UNROLL = 4;
    __shared__ float sv[NT * VEC];
    __shared__ int si[NT * VEC];
    const int tid = threadIdx.x;
    const long long o = blockIdx.x / (unsigned int)segs;
    const int seg = (int)(blockIdx.x - (unsigned int)o * (unsigned int)segs);
    const int r0 = seg * r_per_seg;
    const int r1 = r0 + r_per_seg < red ? r0 + r_per_seg : red;
    const long long n = (long long)(r1 - r0) * inner;             // elements of this block
    const int P = R * inner;
    const size_t first = ((size_t)o * (size_t)red + (size_t)r0) * (size_t)inner;
    const unsigned char* const at0 = (const unsigned char*)X + first * ES;
    const bool whole = P % VEC == 0;
    const int lead = whole ? (int)((size_t)at0 & 15u) / ES : 0;
    const int f0 = tid * VEC - lead;                              // this lane's first element of period 0
    const bool mine = tid * VEC < P;
    const int periods = (int)((n + lead + P - 1) / P);
    // periods before this one lie inside the block to the last chunk (but for the first one, which may start before it)
    const int full_end = whole ? periods - 1 : periods - 2;

    float bv[VEC];
    int bk[VEC];                                                  // period of the best element, -1: none seen
#pragma unroll
    for (int e = 0; e < VEC; ++e) { bv[e] = kNegInf; bk[e] = -1; }

    if (mine) {
        auto consume = [&](const u32x4& w, int s, bool ok) __attribute__((always_inline)) {
            float x[VEC];
            unpack<BF16>(w, x);
#pragma unroll
            for (int e = 0; e < VEC; ++e)
                if (ok && (bk[e] < 0 || replaces(x[e], bv[e]))) { bv[e] = x[e]; bk[e] = s; }
        };
        // UNROLL periods, of which the block may hold some of the chunks: their loads together all the same
        auto guarded = [&](int s) __attribute__((always_inline)) {
            u32x4 w[UNROLL];
            bool ok[UNROLL];
#pragma unroll
            for (int u = 0; u < UNROLL; ++u) {
                const long long g = (long long)(s + u) * P + f0;
                ok[u] = g >= 0 && g + VEC <= n;
                w[u] = u32x4{0u, 0u, 0u, 0u};
                if (ok[u]) w[u] = load_chunk<BF16, true>(at0 + g * ES);
            }
#pragma unroll
            for (int u = 0; u < UNROLL; ++u) consume(w[u], s + u, ok[u]);
        };
        guarded(0);                                               // (from here on every slot has seen an element, if there is a fifth period)
        int s = UNROLL;
        const unsigned char* src = at0 + ((long long)s * P + f0) * ES;
        const long long step = (long long)P * ES;
        auto sweeps = [&](auto any_start) __attribute__((always_inline)) {
            for (; s + UNROLL <= full_end; s += UNROLL, src += UNROLL * step) {
                u32x4 w[UNROLL];
#pragma unroll
                for (int u = 0; u < UNROLL; ++u) w[u] = load_chunk<BF16, decltype(any_start)::value>(src + u * step);
#pragma unroll
                for (int u = 0; u < UNROLL; ++u) {
                    float x[VEC];
                    unpack<BF16>(w[u], x);
#pragma unroll
                    for (int e = 0; e < VEC; ++e)
                        if (replaces(x[e], bv[e])) { bv[e] = x[e]; bk[e] = s + u; }
                }
            }
        };
        if (whole) sweeps(std::false_type{});
        else sweeps(std::true_type{});
        for (; s < periods; s += UNROLL) guarded(s);
        // chunks that the block's ends cut, one element per load: this lane's first one, and its last
        auto cut = [&](int s) __attribute__((always_inline)) {
            const long long g = (long long)s * P + f0;
            if ((g >= 0 && g + VEC <= n) || g + VEC <= 0 || g >= n) return;
            float x[VEC];
#pragma unroll
            for (int e = 0; e < VEC; ++e) {                       // (an element there is in any case in place of one that is not)
                const long long ge = g + e < 0 ? 0 : g + e < n ? g + e : n - 1;
                x[e] = load_one<BF16>(at0, (size_t)ge);
            }
#pragma unroll
            for (int e = 0; e < VEC; ++e)
                if (g + e >= 0 && g + e < n && beats(x[e], s, bv[e], bk[e] < 0 ? kNoPos : bk[e])) { bv[e] = x[e]; bk[e] = s; }
        };
        cut(0);
        if (periods > 1) cut(periods - 1);
        if (!whole && periods > 2) cut(periods - 2);              // (its last chunk reaches into the last period)
        // element f of the period (those before the block: of the period before) is r number f / inner, position f % inner
        int q = f0 < 0 ? -((-f0 + inner - 1) / inner) : f0 / inner, i = f0 - q * inner;
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            const int f = f0 + e, k = f < 0 ? f + P : f;
            if (k < P) {
                sv[k] = bv[e];
                si[k] = bk[e] < 0 ? kNoPos : r0 + bk[e] * R + q;
            }
            if (++i == inner) { i = 0; ++q; }
        }
    }
    __syncthreads();
    for (int rows = R; rows > 1;) {
        const int left = (rows + 3) / 4, n_left = left * inner, n_rows = rows * inner;
        for (int k = tid; k < n_left; k += NT) {
            float v = sv[k];
            int p = si[k];
#pragma unroll
            for (int j = 1; j < 4; ++j) {
                const int kk = k + j * n_left;
                if (kk < n_rows) {
                    const float ov = sv[kk];
                    const int op = si[kk];
                    if (beats(ov, op, v, p)) { v = ov; p = op; }
                }
            }
            sv[k] = v;
            si[k] = p;
        }
        rows = left;
        __syncthreads();
    }
    for (int k = tid; k < inner; k += NT) {
        if (segs == 1) {
            store_one<BF16>(out, (size_t)o * inner + k, sv[k]);
            if (idx) idx[(size_t)o * inner + k] = si[k];
        } else {
            const size_t at = ((size_t)o * segs + seg) * (size_t)inner + k;
            pv[at] = sv[k];
            pi[at] = si[k];
        }
    }
}

// ---------------------------------------------------------------------------------
// inner > 1 and red x inner <= 128: the block of one outer index is smaller than a wave's
// worth of work.  A workgroup takes Q = 256 / (red x inner) outer indices: its threads load
// the Q blocks (contiguous in memory) into LDS, one element each, then one thread per output
// scans its red values in order.
template <bool BF16>
__global__ __launch_bounds__(256) void reduce_max_tiny_block_kernel(const void* __restrict__ X, void* __restrict__ out,
                                                                    int* __restrict__ idx, long long outer, int red, int inner)
{
    __shared__ float vals[256];
    const int tid = threadIdx.x;
    const int block = red * inner, Q = 256 / block;
    const long long o0 = (long long)blockIdx.x * Q;
    const int q_mine = tid / block;
    if (q_mine < Q && o0 + q_mine < outer) vals[tid] = load_one<BF16>(X, (size_t)o0 * (size_t)block + (size_t)tid);
    __syncthreads();
    const int q = tid / inner, i = tid - q * inner;
    if (q < Q && o0 + q < outer) {
        const float* mine = vals + q * block + i;
        float v = mine[0];
        int p = 0;
        for (int r = 1; r < red; ++r) {
            const float x = mine[r * inner];
            if (replaces(x, v)) { v = x; p = r; }
        }
        const size_t at = (size_t)(o0 + q) * (size_t)inner + (size_t)i;
        store_one<BF16>(out, at, v);
        if (idx) idx[at] = p;
    }
}

// Second pass: one thread per output, the segment results taken in order.
template <bool BF16>
__global__ __launch_bounds__(256) void reduce_max_finish_kernel(const float* __restrict__ pv, const int* __restrict__ pi,
                                                                void* __restrict__ out, int* __restrict__ idx,
                                                                long long outer, long long inner, int segs)
{
    const long long t = (long long)blockIdx.x * 256 + threadIdx.x;
    if (t >= outer * inner) return;
    const long long o = t / inner, i = t - o * inner;
    const size_t base = (size_t)o * segs * (size_t)inner + (size_t)i;
    float v = pv[base];
    int p = pi[base];
    for (int s = 1; s < segs; ++s) {
        const float ov = pv[base + (size_t)s * (size_t)inner];
        const int op = pi[base + (size_t)s * (size_t)inner];
        if (beats(ov, op, v, p)) { v = ov; p = op; }
    }
    store_one<BF16>(out, (size_t)t, v);
    if (idx) idx[t] = p;
}

// The same with one wave per output, for many segments (few outputs, long rows): the lanes
// take every 64th segment, then the pairs are combined across the lanes.  The combine picks
// by (value, then earlier position), so the order it is applied in does not matter.
template <bool BF16>
__global__ __launch_bounds__(256) void reduce_max_finish_wave_kernel(const float* __restrict__ pv, const int* __restrict__ pi,
                                                                     void* __restrict__ out, int* __restrict__ idx,
                                                                     long long outer, long long inner, int segs)
{
    const int lane = threadIdx.x & 63;
    const long long t = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (t >= outer * inner) return;          // whole waves leave together
    const long long o = t / inner, i = t - o * inner;
    const size_t base = (size_t)o * segs * (size_t)inner + (size_t)i;
    float v = kNegInf;
    int p = kNoPos;
    for (int s = lane; s < segs; s += 64) {
        const float ov = pv[base + (size_t)s * (size_t)inner];
        const int op = pi[base + (size_t)s * (size_t)inner];
        if (beats(ov, op, v, p)) { v = ov; p = op; }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        const float ov = __shfl_xor(v, off, 64);
        const int op = __shfl_xor(p, off, 64);
        if (beats(ov, op, v, p)) { v = ov; p = op; }
    }
    if (lane == 0) {
        store_one<BF16>(out, (size_t)t, v);
        if (idx) idx[t] = p;
    }
}

// Workgroups a launch is cut into when the outputs alone give fewer: two per CU for fp32, four
// for bf16 (more vector ALU work per byte).  More, shorter segments stream worse -- measured on
// 1 GiB tensors, fp32 strided 6800 GB/s at 512 workgroups, 6500 at 1024, 6370 at 2048; bf16
// strided 5080 / 6450 / 5970; fp32 long rows 6940 / 6670 / 6620.
constexpr int target_workgroups(int dtype) { return dtype == DT_BF16 ? 1024 : 512; }
constexpr int kWaveFinishMinSegs = 16;
// Rows are held in registers up to so many chunks by some lanes of a wave or all of them, by a workgroup of 256, eight chunks a lane at most
// (300 MB of fp32 rows of 2112 elements 43 us so, 63 swept by a wave each; bf16 of 8192 44 and 50), and by 512 threads, sixteen chunks a lane (bf16
// [2048, 50257] 33 us so, 37 swept by 256; fp32 rows of 14400 36 and 39).  With too few rows for every CU 1024 threads hold
// as many, also where rows would be cut into segments: the second pass is a launch of its own (bf16 [128, 50257] 9.5 us
// so, 5.8 here; [400, 65536] 13.4 and 9.7; but [1000, 24001], one segment, 9.1 and 10.4).  So they do for fp32 rows of 3072 to 6400 chunks, unless
// their last one is less than half used: 512 threads keep more rows under way than the memory takes well (600 MB of rows of 16384 elements 94 us, 89 so,
// 20480 89 and 88; 16448 93 and 95, 28672 90.6 and 91.2).
constexpr long long kHeldWave = 512, kHeldWorkgroup = 2048, kHeldMost = 8192;
constexpr long long kSmallInner = 64;             // inner dimensions up to this: the flattened-sweep kernel
constexpr long long kTinyBlock = 128;             // red x inner up to this: several outer indices per workgroup

// Strided reductions (inner > 1) that reduce_max_block_kernel leaves to the kernels before it
ReducePlan plan_strided(long long outer, long long red, long long inner, int dtype, bool x_aligned)
{
    ReducePlan pl{};
    const int vec16 = dtype == DT_BF16 ? 8 : 4;
    if (inner <= kSmallInner) {
        // one wave per (outer index, segment); group = 0 marks this kernel
        pl.vec = 1;
        pl.group = 0;
        pl.tiles_i = 1;
        pl.segs = 1;
        const long long waves = 4LL * target_workgroups(dtype);
        if (outer < waves) {
            const long long want = (waves + outer - 1) / outer;
            const long long sweep = 64 / inner;                                  // r per sweep
            const long long most = red / (8 * sweep) > 0 ? red / (8 * sweep) : 1;   // eight sweeps per segment at least
            pl.segs = (int)(want < most ? want : most);
        }
        pl.per_seg = (int)((red + pl.segs - 1) / pl.segs);
        pl.segs = (int)((red + pl.per_seg - 1) / pl.per_seg);
        pl.blocks = (outer * pl.segs + 3) / 4;
    } else {
        pl.unaligned = !(x_aligned && inner % vec16 == 0);
        // One element per load for unaligned rows while the problem is small: the chip is not full then, and
        // 64 VEC positions per workgroup leave fewer and longer ones (fp32 [53, 67, 845] 10.1 us, in chunks 15.3;
        // bf16 [580, 101, 83] 10.0 and 15.4); bf16 also with few positions per row, where most lanes have
        // no chunk ([484, 279, 102] 19.3 and 22.9).  Of 20000 unaligned shapes 0.8 % stay more than
        // 5 % behind one element per load everywhere, without these lines 5 %; the mean is 1.25 (bf16) and 1.38
        // (fp32) times as fast as with one element everywhere.
        const long double elements = (long double)outer * red * inner;
        const bool single = pl.unaligned && (elements < (dtype == DT_BF16 ? 1.0e7L : 4.0e6L) ||
                                             (dtype == DT_BF16 && inner <= 128 && red < 512));
        pl.vec = single ? 1 : vec16;
        pl.group = 256;
        pl.tiles_i = (int)((inner + 64 * pl.vec - 1) / (64 * pl.vec));
        const long long wg0 = outer * pl.tiles_i;
        pl.segs = 1;
        if (wg0 < target_workgroups(dtype)) {
            const long long want = (target_workgroups(dtype) + wg0 - 1) / wg0;
            // eight r per wave at least; unaligned chunks sixteen, fp32 ones (less work each) thirty-two, else the second pass
            // costs more than the segments give (fp32 [42, 72, 1901]: 13.7 us in one pass, 18.5 in two; [11, 135, 2959] 10.5
            // and 15.8; bf16 [59, 254, 438], 26.9 and 16.0)
            const long long least = !pl.unaligned || single ? 32 : dtype == DT_BF16 ? 64 : 128;
            const long long most = red / least > 0 ? red / least : 1;
            pl.segs = (int)(want < most ? want : most);
        }
        pl.per_seg = (int)((red + pl.segs - 1) / pl.segs);
        pl.segs = (int)((red + pl.per_seg - 1) / pl.per_seg);
        pl.blocks = wg0 * pl.segs;
    }
    pl.partial_elems = pl.segs > 1 ? (size_t)outer * pl.segs * (size_t)inner : 0;
    return pl;
}

// The workgroups and the periods of reduce_max_block_kernel (the plan's `group` is minus its threads, `tiles_i` the r of a period),
// where that kernel is the faster one.  What decides it (calls queued one after the other; of 4500 drawn shapes 1409 are more than a twentieth faster than
// without this kernel, 1.59 times in the mean, five are more than a tenth slower, 0.88 the worst; the figures: the other kernels' time / this one's):
//  * A workgroup starts, ends and combines its lanes once per block (or segment): many small blocks are not for it.  Of 512 blocks and more
//    it takes fp32 ones from 14 bytes per block of them on, 64 KB at most ([9015, 359, 7] 0.65, [1436, 3222, 3] 1.37), 256 KB where inner is over 64
//    ([7361, 20, 207] 0.66, up to 1.66 from there); bf16 ones, which a wave reads element by element, from 2 KB, 8 KB of 1024 and more ([976, 21, 25] 0.67,
//    [570, 830, 2] 1.52), where lanes of the strided kernel read them 32 KB, and there not if these are mostly at work ([1430, 421, 415] 0.80).
//  * Fewer blocks of up to 256 KB: 1024 threads a block and no second pass, instead of segments and one.  A launch is 3 us, a block of 50 KB as
//    long, so the line is at a size of block that grows with all of the input, which the two launches have to read as well (bf16 [249, 461, 63] 2.35, fp32
//    [5, 8632, 7] 0.58; [77, 2865, 3] 1.2).  Where the other kernels make no segments theirs is one launch too and the faster one throughout
//    (bf16 [261, 55, 285] 0.45).
//  * Fewer, larger blocks in segments: two launches either way, from 3 (bf16, inner up to 64) to 36 MB on ([14, 2533, 47] fp32 0.81, [178, 3508, 25]
//    1.62); with inner over 64 where at most half of the strided kernel's lanes are at work in fp32 ([16, 19619, 244] 0.96, [28, 49714, 67] 1.91), for
//    bf16 also beyond unless the blocks are over 80, where that kernel has the workgroups that it needs ([111, 1589, 413] 0.84, [29, 22832, 138] 2.12).
// Segments: 512 workgroups, or 768 or 1024 where these are a whole number for every CU and 512 are not; four periods at
// least, and never more of them than the kernels before this one take, so that no call needs more workspace than with those. Where they take
// fewer than 512 workgroups would be, they are the faster ones by themselves: of 70 such shapes 0.64 to 1.08 of the time here with the segments
// they take, 0.7 on average (fp32 [240, 218, 479] none, bf16 [5, 4283, 282] 41: 11.1 us, 14.5 here), and no slower than with more of them here.
constexpr long long kOneLaunchBytes = 256 << 10;

// pl: the plan of the kernels before this one, left as it is where they are faster -- unless `anywhere`, with which it is left only where this kernel
// does not go.
void plan_block(ReducePlan& pl, long long outer, long long red, long long inner, int dtype, bool anywhere)
{
    const long long es = dtype == DT_BF16 ? 2 : 4, vec = 16 / es;
    const long long bytes = red * inner * es, lanes = 64 * vec;
    const bool bf16 = dtype == DT_BF16, waves = inner <= kSmallInner;      // (waves: the other kernel is the one with a wave per segment)
    const double all = 1.0e-6 * (double)outer * (double)bytes;
    const double busy = (double)inner / (double)((inner + lanes - 1) / lanes * lanes);      // share of the strided kernel's lanes that have positions
    const bool one_launch = outer < 512 && bytes <= kOneLaunchBytes;
    if (one_launch ? inner > 512 * vec || (inner > 128 * vec && red < 64) : inner > 128 * vec) return;
    if (anywhere) {
        // (whatever it takes)
    } else if (one_launch) {
        if (pl.segs == 1) return;
        if (outer > 256) { if (!bf16 || !waves || all < 3.0) return; }
        else if ((double)bytes > 1024.0 * (bf16 ? 13.0 + (waves ? 17.0 : 10.0) * all : 42.0 + 4.5 * all)) return;
    } else if (outer >= 512) {
        const long long least = bf16 ? (waves ? (outer < 1024 ? 2 : 8) : inner <= lanes ? 32 : 8) * 1024 : waves ? std::min(14 * outer, 65536LL) : 256 * 1024;
        if (bytes < least || (bf16 && !waves && inner <= lanes && busy > 0.7)) return;
    } else if (waves) {
        if (all < (bf16 ? 3.0 : pl.segs >= 650 ? 2.5 : 32.0)) return;
    } else if (bf16 ? all < 20.0 || (outer > 80 && busy > 0.7) : all < 36.0 || busy > 0.5) {
        return;
    }
    const long long nt = one_launch ? 1024 : 256;
    long long R = nt * vec / inner;
    const long long common = (inner & -inner) < vec ? (inner & -inner) : vec;      // (greatest common divisor: vec is a power of two)
    if (R >= 4 * (vec / common)) R -= R % (vec / common);
    if (!anywhere && !one_launch && inner > 64 * vec && 4 * R * inner < 3 * nt * vec) return;
    long long segs = 1;
    if (!one_launch && outer < 512) {
        const long long periods = red / (4 * R), wanted = 512 / outer < periods ? 512 / outer : periods;
        if (!anywhere && wanted > pl.segs) return;
        const long long most = periods < pl.segs ? periods : pl.segs;
        double best = 0.0;
        for (long long target = 512; target <= 1024; target += 256) {
            const long long n = target / outer < most ? target / outer : most;
            const double filled = (double)(n * outer) / (double)target;
            if (n >= 1 && filled > best + 0.05) { best = filled; segs = n; }
        }
        if (!anywhere && inner > 64 * vec && segs == pl.segs && segs * outer < 448) return;
    }
    pl.unaligned = false;
    pl.vec = (int)vec;
    pl.group = (int)-nt;
    pl.per_seg = (int)((red + segs - 1) / segs);
    pl.segs = (int)((red + pl.per_seg - 1) / pl.per_seg);
    pl.tiles_i = (int)(R < pl.per_seg ? R : pl.per_seg);
    pl.blocks = outer * pl.segs;
    pl.partial_elems = pl.segs > 1 ? (size_t)outer * pl.segs * (size_t)inner : 0;
}

}  // namespace

ReducePlan plan_reduce_max(long long outer, long long red, long long inner, int dtype, bool x_aligned)
{
    ReducePlan pl{};
    const int es = dtype == DT_BF16 ? 2 : 4;
    const int vec16 = 16 / es;
    if (inner == 1) {
        pl.unaligned = !(x_aligned && red % vec16 == 0);
        pl.vec = red < vec16 ? 1 : vec16;
        const long long all = (red + pl.vec - 1) / pl.vec;
        const bool few = outer <= 256 || (outer < target_workgroups(dtype) && all >= 2 * kHeldWorkgroup);
        if (all <= kHeldMost) {
            // The fewest lanes that hold the row: with two chunks each, so that short rows are read in pieces of 128 bytes, from eight lanes on
            // with four (fp32 rows of 64 elements 50 us on four lanes, 44 on eight; bf16 of 520 47 on 32 lanes, 72 on 64).
            int g = 1;
            if (all > kHeldWorkgroup) g = few || (dtype == DT_F32 && all >= 3072 && all <= 6400 && (all - 1) % 1024 >= 512) ? 1024 : 512;
            else if (all > kHeldWave) g = 256;
            else if (pl.vec > 1) while ((all <= 16 ? 2 : 4) * g < all && g < 64) g *= 2;
            pl.group = g;
            pl.held = true;
            pl.segs = 1;
            pl.per_seg = (int)((all + g - 1) / g);
            pl.tiles_i = 1;
            pl.blocks = g > 64 ? outer : (outer + 256 / g - 1) / (256 / g);
            pl.partial_elems = 0;
            return pl;
        }
        const long long nch = red / pl.vec;
        pl.group = 256;
        pl.segs = 1;
        if (outer < target_workgroups(dtype)) {
            const long long want = (target_workgroups(dtype) + outer - 1) / outer;
            const long long most = nch / (256 * 8) > 0 ? nch / (256 * 8) : 1;   // eight sweeps per segment at least
            pl.segs = (int)(want < most ? want : most);
        }
        pl.per_seg = (int)((nch + pl.segs - 1) / pl.segs);
        pl.segs = (int)((nch + pl.per_seg - 1) / pl.per_seg);
        pl.blocks = outer * pl.segs;
        pl.tiles_i = 1;
    } else if (red * inner <= kTinyBlock) {
        // several outer indices per workgroup; group = -1 marks this kernel
        pl.vec = 1;
        pl.group = -1;
        pl.tiles_i = 1;
        pl.segs = 1;
        pl.per_seg = (int)red;
        const long long q = 256 / (red * inner);
        pl.blocks = (outer + q - 1) / q;
    } else {
        pl = plan_strided(outer, red, inner, dtype, x_aligned);
        plan_block(pl, outer, red, inner, dtype, false);
        return pl;
    }
    pl.partial_elems = pl.segs > 1 ? (size_t)outer * pl.segs * (size_t)inner : 0;
    return pl;
}

ReducePlan plan_reduce_max_blocks(long long outer, long long red, long long inner, int dtype, bool x_aligned)
{
    if (inner == 1 || red * inner <= kTinyBlock) return {};
    ReducePlan pl = plan_strided(outer, red, inner, dtype, x_aligned);
    plan_block(pl, outer, red, inner, dtype, true);
    return pl.group <= -256 ? pl : ReducePlan{};
}

namespace {

template <bool BF16, int VEC, int FORM, int G, int U = 8>
void launch_held(const ReducePlan& pl, const void* X, void* out, int* idx, long long outer, int red, hipStream_t s)
{
    if (pl.per_seg != U) {
        if constexpr (U > (G == 512 ? 5 : G > 64 ? 3 : 1)) launch_held<BF16, VEC, FORM, G, U - 1>(pl, X, out, idx, outer, red, s);
        return;
    }
    int lg = 0;
    while ((1 << lg) < pl.group) ++lg;
    hipLaunchKernelGGL((reduce_max_held_rows_kernel<BF16, VEC, FORM, U, G>), dim3((unsigned int)pl.blocks), dim3(G > 64 ? G : 256), 0, s, X, out, idx,
                       outer, red, lg);
}

template <bool BF16>
void launch_held(const ReducePlan& pl, const void* X, void* out, int* idx, long long outer, int red, hipStream_t s)
{
    constexpr int VEC = Elem<BF16>::VEC, OFF = BF16 ? LEAD : ANY;
    if (pl.vec == 1) launch_held<BF16, 1, ALIGNED, 64, VEC - 1>(pl, X, out, idx, outer, red, s);
    else if (pl.group <= 64) {
        if (pl.unaligned) launch_held<BF16, VEC, ANY, 64>(pl, X, out, idx, outer, red, s);
        else launch_held<BF16, VEC, ALIGNED, 64>(pl, X, out, idx, outer, red, s);
    } else if (pl.group == 256) {
        if (pl.unaligned) launch_held<BF16, VEC, OFF, 256>(pl, X, out, idx, outer, red, s);
        else launch_held<BF16, VEC, ALIGNED, 256>(pl, X, out, idx, outer, red, s);
    } else if (pl.group == 512) {
        if (pl.unaligned) launch_held<BF16, VEC, OFF, 512, 16>(pl, X, out, idx, outer, red, s);
        else launch_held<BF16, VEC, ALIGNED, 512, 16>(pl, X, out, idx, outer, red, s);
    } else {
        if (pl.unaligned) launch_held<BF16, VEC, OFF, 1024>(pl, X, out, idx, outer, red, s);
        else launch_held<BF16, VEC, ALIGNED, 1024>(pl, X, out, idx, outer, red, s);
    }
}

}  // namespace

hipError_t launch_reduce_max(const ReducePlan& pl, const void* X, void* out, int* idx, float* pv, int* pi,
                             long long outer, long long red, long long inner, int dtype, hipStream_t s)
{
    if (pl.blocks <= 0 || pl.blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    const dim3 grid((unsigned int)pl.blocks), block(256);
    const bool bf = dtype == DT_BF16;
    if (pl.held) {
        if (bf) launch_held<true>(pl, X, out, idx, outer, (int)red, s);
        else launch_held<false>(pl, X, out, idx, outer, (int)red, s);
    } else if (inner > 1 && pl.group <= -256) {
#define PGK_BLOCK(BF, NT) \
    hipLaunchKernelGGL((reduce_max_block_kernel<BF, NT>), grid, dim3(NT), 0, s, X, out, idx, pv, pi, (int)red, (int)inner, pl.segs, pl.per_seg, pl.tiles_i)
        if (bf) { if (pl.group == -256) PGK_BLOCK(true, 256); else PGK_BLOCK(true, 1024); }
        else { if (pl.group == -256) PGK_BLOCK(false, 256); else PGK_BLOCK(false, 1024); }
#undef PGK_BLOCK
    } else if (inner > 1 && pl.group == -1) {
        if (bf) hipLaunchKernelGGL(reduce_max_tiny_block_kernel<true>, grid, block, 0, s, X, out, idx, outer, (int)red, (int)inner);
        else hipLaunchKernelGGL(reduce_max_tiny_block_kernel<false>, grid, block, 0, s, X, out, idx, outer, (int)red, (int)inner);
    } else if (inner > 1 && pl.group == 0) {
        if (bf) hipLaunchKernelGGL(reduce_max_small_inner_kernel<true>, grid, block, 0, s, X, out, idx, pv, pi, outer, (int)red, (int)inner, pl.segs, pl.per_seg);
        else hipLaunchKernelGGL(reduce_max_small_inner_kernel<false>, grid, block, 0, s, X, out, idx, pv, pi, outer, (int)red, (int)inner, pl.segs, pl.per_seg);
    } else if (inner == 1) {
        // (sweeps at a time: two, but of fp32 four with at most two workgroups a CU, where two are too few loads under way -- [512, 200000]
        // 70 us, 59, [16, 2^24] 175 and 151 --, and with more than four; between, [396, 1077376] takes 250 us with two, 274 with
        // four.  bf16 [1195, 101129] 40.7 and 41.4)
        const bool two = pl.blocks > 512 && pl.blocks <= 1024;
#define PGK_ROWS(BF, ENDS, N) \
    hipLaunchKernelGGL((reduce_max_rows_kernel<BF, ENDS, N>), grid, block, 0, s, X, out, idx, pv, pi, (int)red, pl.segs, pl.per_seg)
        if (bf) { if (pl.unaligned) PGK_ROWS(true, true, 2); else PGK_ROWS(true, false, 2); }
        else if (two) { if (pl.unaligned) PGK_ROWS(false, true, 2); else PGK_ROWS(false, false, 2); }
        else { if (pl.unaligned) PGK_ROWS(false, true, 4); else PGK_ROWS(false, false, 4); }
#undef PGK_ROWS
    } else {
#define PGK_COLS(BF, VEC, UN) \
    hipLaunchKernelGGL((reduce_max_cols_kernel<BF, VEC, UN>), grid, block, 0, s, X, out, idx, pv, pi, outer, (int)red, inner, pl.tiles_i, pl.segs, pl.per_seg)
        if (bf) { if (pl.vec == 1) PGK_COLS(true, 1, true); else if (pl.unaligned) PGK_COLS(true, 8, true); else PGK_COLS(true, 8, false); }
        else { if (pl.vec == 1) PGK_COLS(false, 1, true); else if (pl.unaligned) PGK_COLS(false, 4, true); else PGK_COLS(false, 4, false); }
#undef PGK_COLS
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || pl.segs == 1) return e;
    const long long outs = outer * inner;
    if (pl.segs >= kWaveFinishMinSegs) {
        const long long wb = (outs + 3) / 4;
        if (wb > 0x7fffffffLL) return hipErrorInvalidValue;
        if (bf) hipLaunchKernelGGL(reduce_max_finish_wave_kernel<true>, dim3((unsigned int)wb), block, 0, s, pv, pi, out, idx, outer, inner, pl.segs);
        else hipLaunchKernelGGL(reduce_max_finish_wave_kernel<false>, dim3((unsigned int)wb), block, 0, s, pv, pi, out, idx, outer, inner, pl.segs);
        return hipGetLastError();
    }
    const long long fb = (outs + 255) / 256;
    if (fb > 0x7fffffffLL) return hipErrorInvalidValue;
    if (bf) hipLaunchKernelGGL(reduce_max_finish_kernel<true>, dim3((unsigned int)fb), block, 0, s, pv, pi, out, idx, outer, inner, pl.segs);
    else hipLaunchKernelGGL(reduce_max_finish_kernel<false>, dim3((unsigned int)fb), block, 0, s, pv, pi, out, idx, outer, inner, pl.segs);
    return hipGetLastError();
}

}  // namespace pgk
