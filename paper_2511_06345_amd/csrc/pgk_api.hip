// C-ABI layer of libpgk: argument validation (host only, before any HIP call),
// choice of kernel path and launch geometry, and the layout of the caller's workspace.
// The library allocates no device memory and keeps no state between calls.
// The contract of every entry point is documented in include/pgk.h.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <mutex>

#include "../../include/pgk.h"
#include "pgk_kernels.h"

// The fixed workspace of pgk_gemm_fused_static (device memory; see static_scratch_of_current_device).
static __device__ __align__(256) unsigned char scratch[(size_t)4 << 20];

namespace {

using pgk::GemmArgs;

constexpr int64_t kMaxDim = 0x7fffffffLL;
constexpr int kNumCUs = 256;          // MI355X
// Shortest slice of an automatic split, in K tiles: below that the second pass and launch cost
// more than the shorter loop saves.  16; for bf16, whose K tile takes half as long as an fp32
// one, 32 once the small-tile grid has 96 workgroups (with slices of 16: 1024 x 2048 x 2048 27 us
// in two slices, 20 us in one, 1536 x 1536 x 4096 45 us in four, 41 us in two; but 768 x 768 x 3072,
// 36 tiles, 22 us in three and 32 us in one; fp32 512 x 512 x 1024 18 us in two, 22 us in one).
int min_steps_per_slice(int dtype, long double small_tiles) { return dtype == PGK_DTYPE_BF16 && small_tiles >= 96 ? 32 : 16; }
constexpr size_t kAutoSplitMaxWorkspace = (size_t)256 << 20;   // workspace pgk_gemm_fused may ask for an automatic split
constexpr int kMaxAutoSplits = 32;
constexpr int64_t kLongKSteps = 512;

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

int validate_common(const void* A, const void* B, const void* C, int64_t M, int64_t N, int64_t K,
                    int64_t batch, int act, int dtype)
{
    if (!A || !B || !C) return PGK_ERR_INVALID_ARG;
    if (M <= 0 || N <= 0 || K <= 0 || batch <= 0) return PGK_ERR_INVALID_ARG;
    if (act < PGK_ACT_NONE || act > PGK_ACT_SILU) return PGK_ERR_INVALID_ARG;
    if (dtype != PGK_DTYPE_F32 && dtype != PGK_DTYPE_BF16) return PGK_ERR_INVALID_ARG;
    if (M > kMaxDim || N > kMaxDim || K > kMaxDim || batch > kMaxDim) return PGK_ERR_UNSUPPORTED;
    const long double lim = 4.6e18L;  // 2^62
    if ((long double)batch * M * N >= lim || (long double)batch * M * K >= lim ||
        (long double)batch * K * N >= lim)
        return PGK_ERR_UNSUPPORTED;
    return PGK_OK;
}

int kstep_of(int dtype) { return pgk::mfma_tile_shape(dtype, false).bk; }

// Split geometry shared by the workspace query and the launch: slice length L
// and the number of non-empty slices.
struct SplitPlan { int splits; int k_slice; };

size_t round_up256(size_t v) { return (v + 255) / 256 * 256; }
int64_t chunk_elems(int dtype) { return dtype == PGK_DTYPE_BF16 ? 8 : 4; }
int64_t round_up64(int64_t v, int64_t a) { return (v + a - 1) / a * a; }

// Outputs with at most 32 columns or rows: the skinny tiles (narrow 128 x 32, flat 32 x 128), on
// which such a product stays bound by the stream of its large operand instead of by matrix work
// on padding (bf16 16384 x 16 x 16384: 137 us on 128 x 128 tiles).  The narrow tile exists for a
// transposed B only; a plain B of so few columns is small and is transposed first (see route_for).
// -1: not skinny.
int skinny_tile_kind(int64_t M, int64_t N)
{
    if (M <= 32 && N > 32) return pgk::TILE_FLAT;
    if (N <= 32 && M > 32) return pgk::TILE_NARROW;
    if (M <= 32 && N <= 32) return pgk::TILE_FLAT;
    return -1;
}

// Operand rows that would start off 4-byte boundaries (bf16: an odd K, or an odd N for a plain B), which
// the direct-to-LDS copies do not take.
struct OddRows { bool a, b; };
OddRows odd_rows(int64_t K, int dtype, bool b_trans, int64_t ldb)
{
    const int64_t es = dtype == PGK_DTYPE_BF16 ? 2 : 4;
    return {(K * es) % 4 != 0, ((b_trans ? K : ldb) * es) % 4 != 0};
}

// Whether there is a kernel that copies such operands through registers (pgk_gemm_mfma_reg.hip): skinny tiles have no such
// instance, and problems of less than 2^25 multiply-adds keep to the workspace they have always asked for.
// (What it costs against padded copies: reg_copies_pay.)
bool reg_copies_exist(int64_t M, int64_t N, int64_t K)
{
    return skinny_tile_kind(M, N) < 0 && (long double)M * N * K >= 33554432.0L;
}

// What the matrix-core kernels take as it is: operand rows that start on 4-byte boundaries (K
// elements for A and a transposed B; the row length ldb of a plain B, which is N unless the
// caller has padded it), bf16 rows on any element where reg_copies_exist.  M, N and K need not be tile multiples, and the
// output rows may have any length.  An output below 16 x 16 is left to the bounds-checked kernel, which wastes less, unless K is
// long (then the matrix-core route splits the K range over the chip).
bool mfma_shape_ok(int64_t M, int64_t N, int64_t K, int dtype, bool b_trans = false, int64_t ldb = 0)
{
    const pgk::TileShape t = pgk::mfma_tile_shape(dtype, false);
    const int64_t es = dtype == PGK_DTYPE_BF16 ? 2 : 4;
    if (!ldb) ldb = b_trans ? K : N;
    const OddRows odd = odd_rows(K, dtype, b_trans, ldb);
    if ((odd.a || odd.b) && !reg_copies_exist(M, N, K)) return false;
    if (M < 16 && N < 16 && K < 1024) return false;
    // per-lane 32-bit byte offsets inside one tile
    if ((int64_t)t.bm * K * es >= (1LL << 32)) return false;
    if ((b_trans ? (int64_t)t.bn * K : (int64_t)t.bk * ldb) * es >= (1LL << 32)) return false;
    return true;
}

// The slices of a split call (0: the fused call's own plan) and the tile that an automatic count comes with (-1: by the grid).
// no_copies: registers wherever there is a kernel for them (a workspace without room for padded copies)
struct Slices { int count, kind; bool no_copies; };

bool reg_copies_pay(int64_t M, int64_t N, int64_t K, int64_t batch, int dtype, bool b_trans, Slices slices);

// Odd rows that no kernel takes as they are, or that are cheaper copied: the operands are first copied into buffers with
// rows padded with zeros to whole 16-byte chunks.  Worth it from about 64^3 multiply-adds on.
bool needs_packing(int64_t M, int64_t N, int64_t K, int64_t batch, int dtype, bool b_trans, Slices slices)
{
    const OddRows odd = odd_rows(K, dtype, b_trans, N);
    return (odd.a || odd.b) && !(reg_copies_exist(M, N, K) && (slices.no_copies || reg_copies_pay(M, N, K, batch, dtype, b_trans, slices)));
}

// The dimensions the kernels see for a problem that is packed first: K and the row length of B,
// rounded up to whole chunks where they are odd.  pack = false: the problem is taken as it is (aligned already, or
// too small or too large for this to pay).
// transpose_b: a plain B of at most 32 columns under more than 32 rows of output is copied in
// transposed form, [N][k], for the narrow tile; the kernels then see a transposed B (b_trans).
struct PackDims { bool pack; int64_t k, ldb; bool transpose_b; bool b_trans; };

// misaligned: A or B does not start on a 16-byte boundary; the copies do (pack_operands copies
// whichever operand needs it), and their rows are whole chunks.
PackDims pack_dims(int64_t M, int64_t N, int64_t K, int64_t batch, int dtype, bool b_trans, Slices slices, bool misaligned = false)
{
    const PackDims as_is{false, K, 0, false, b_trans};
    const bool transpose_b = !b_trans && skinny_tile_kind(M, N) == pgk::TILE_NARROW;
    if (!transpose_b && !misaligned && !needs_packing(M, N, K, batch, dtype, b_trans, slices)) return as_is;
    if ((long double)M * N * K < 262144.0L) return as_is;
    const int64_t epc = chunk_elems(dtype), es = dtype == PGK_DTYPE_BF16 ? 2 : 4;
    PackDims d{true, ((K * es) % 4 || misaligned) ? round_up64(K, epc) : K, 0, transpose_b, b_trans || transpose_b};
    // (a plain B is copied in every such case; so is a B that is transposed, with rows of whole chunks)
    d.ldb = transpose_b ? round_up64(d.k, epc) : d.b_trans ? d.k : round_up64(N, epc);
    if (d.k > kMaxDim || d.ldb > kMaxDim) return as_is;
    if (!mfma_shape_ok(M, N, d.k, dtype, d.b_trans, d.ldb)) return as_is;
    return d;
}

// the plan queries, which do not know the layout of B: does this problem end up on the matrix
// cores, one way or the other, with either layout
bool mfma_route(int64_t M, int64_t N, int64_t K, int dtype)
{
    const Slices fused{0, -1, false};
    return mfma_shape_ok(M, N, K, dtype) || pack_dims(M, N, K, 1, dtype, false, fused).pack ||
           mfma_shape_ok(M, N, K, dtype, true) || pack_dims(M, N, K, 1, dtype, true, fused).pack;
}

// A large tile mostly outside the matrix (skinny M or N): the small tile wastes less matrix work
// and fewer operand loads.  bf16: three quarters empty (between a quarter and a half full the
// half tiles take over; 128 x 65536 x 1024 took 35 us with the large tile, 28 us with either the
// small or the half one).  fp32, which has no half tiles: half empty -- 64 x 65536 x 1024 took
// 146 us with the large tile and 78 us with the small one, 96 x 65536 x 1024 133 and 146 us.
bool large_tile_mostly_empty(int64_t M, int64_t N, int dtype)
{
    const pgk::TileShape big = pgk::mfma_tile_shape(dtype, false);
    const int64_t f = dtype == PGK_DTYPE_BF16 ? 4 : 2;
    return f * M <= big.bm || f * N <= big.bn;
}

// How long a grid of one tile shape takes, in rounds: the chip runs per_cu workgroups per CU
// side by side, a full round of them takes fixed + per_k * K / 1024 (microseconds on the
// measured part; only ratios between shapes are used), and a last, partly filled round with j
// workgroups on its busiest CU takes the share tail[j - 1] of a full one.  Fitted to GEMMs of
// 2560^2 ... 8192^2 outputs with K = 1024 ... 4096 (e.g. bf16 4096^2 x 4096: 256 large tiles 104 us,
// 1024 small ones 122 us, 512 half tiles 114 us; fp32: 1024 large 913 us, 4096 small 965 us).
// The fp32 large tile of these figures, and of the ones beside auto_split and large_tile_mostly_empty, used the fp32
// instruction; in three bf16 terms it takes 0.77 of them, which only auto_tile_kind counts so far.
struct TileCost { int per_cu; double fixed, per_k; double tail[4]; };

TileCost tile_cost(int dtype, int kind)
{
    if (dtype == PGK_DTYPE_BF16) {
        switch (kind) {
        case pgk::TILE_SMALL: return {2, 2.9, 14.3, {0.47, 1.0, 1.0, 1.0}};
        case pgk::TILE_TALL: return {1, 5.8, 12.8, {0.65, 1.0, 1.0, 1.0}};
        case pgk::TILE_WIDE: return {1, 5.7, 13.2, {0.65, 1.0, 1.0, 1.0}};
        default: return {1, 10.0, 22.5, {0.7, 1.0, 1.0, 1.0}};
        }
    }
    if (kind == pgk::TILE_SMALL) return {4, 1.5, 59.9, {0.3, 0.6, 0.75, 1.0}};
    return {1, 3.0, 56.2, {1.0, 1.0, 1.0, 1.0}};
}

// full rounds, and the workgroups on the busiest CU of the last one where that is not full
struct Rounds { double full; int rest; };

Rounds rounds_of(int64_t M, int64_t N, int dtype, int64_t units, int kind)
{
    const pgk::TileShape t = pgk::mfma_tile_shape(dtype, kind);
    const double wgs = (double)((M + t.bm - 1) / t.bm) * (double)((N + t.bn - 1) / t.bn) * (double)units;
    const double slots = (double)kNumCUs * tile_cost(dtype, kind).per_cu;
    const double full = std::floor(wgs / slots);
    return {full, (int)std::ceil((wgs - full * slots) / kNumCUs)};
}

double estimated_rounds_time(int64_t M, int64_t N, int64_t K, int dtype, int64_t units, int kind)
{
    const TileCost c = tile_cost(dtype, kind);
    const Rounds r = rounds_of(M, N, dtype, units, kind);
    return (c.fixed + c.per_k * (double)K / 1024.0) * (r.full + (r.rest > 0 ? c.tail[r.rest - 1] : 0.0));
}

// Automatic choice (splits == 0): slices of at least min_steps_per_slice K steps (shorter ones
// are all prologue and epilogue), at most kMaxAutoSplits of them, and the smallest count that
// gives 2 x 256 workgroups.  The tile the count is made with: a skinny one for skinny outputs,
// else the large one if it can reach 1.5 x 256 workgroups within those limits and is not mostly
// empty, else the small one.
struct AutoPlan { int splits; int kind; };

// fit_round: slices and large tiles are counted so that a grid fits one round where it can (see auto_split).
AutoPlan count_slices(int64_t M, int64_t N, int64_t K, int64_t batch, int dtype, bool fit_round)
{
    const int ks = kstep_of(dtype);
    const int64_t ksteps = (K + ks - 1) / ks;
    auto tiles_of = [&](int kind) {
        const pgk::TileShape t = pgk::mfma_tile_shape(dtype, kind);
        return (long double)((M + t.bm - 1) / t.bm) * ((N + t.bn - 1) / t.bn) * batch;
    };
    // (outputs of at most 64 rows or columns are bound by the stream of their large operand, which
    // more workgroups pull harder on: 16 K tiles per slice for them in any case)
    int64_t s_max = ksteps / ((M <= 64 || N <= 64) ? 16 : min_steps_per_slice(dtype, tiles_of(pgk::TILE_SMALL)));
    if (s_max < 1) s_max = 1;
    if (s_max > kMaxAutoSplits) s_max = kMaxAutoSplits;
    int kind = skinny_tile_kind(M, N);
    if (kind < 0)
        kind = (large_tile_mostly_empty(M, N, dtype) || tiles_of(pgk::TILE_LARGE) * s_max < 1.5L * kNumCUs) ? pgk::TILE_SMALL
                                                                                                          : pgk::TILE_LARGE;
    const long double tiles = tiles_of(kind);
    // (enough slices for two workgroups per CU; four of the fp32 small tile and one of the bf16
    // large tile, which is how many of those fit a CU: a second round of half-length slices does
    // the same matrix work and doubles the partial products -- bf16 1024 x 2048 x 16384 took 100 us
    // in 16 slices and 78 us in 8)
    const long double target = (dtype == PGK_DTYPE_F32 && kind == pgk::TILE_SMALL   ? 4.0L
                                : dtype == PGK_DTYPE_BF16 && kind == pgk::TILE_LARGE ? 1.0L
                                                                                      : 2.0L) * kNumCUs;
    auto slices_for = [&](long double n_tiles, long double goal) {
        int64_t n = 1;
        while (n < s_max && n_tiles * n < 0.95L * goal) ++n;      // (250 tiles: two slices, not three)
        // The goal is also what the chip holds at once (but for skinny tiles): a few workgroups more run as a round of
        // their own, and one slice less, in one round, is done sooner.
        if (fit_round && skinny_tile_kind(M, N) < 0 && n >= 4 && n_tiles * n > goal) --n;
        return n;
    };
    int64_t s = slices_for(tiles, target);
    // Large against small tile once more, now with their slice counts, by the round model (plus
    // what the partial products cost: written and read once, at about 4 TB/s, and a launch): the
    // rule above takes the large tile whenever it can fill the chip, also when its grid then ends
    // in a poorly filled round or needs many more slices (fp32 1536 x 1536 x 8192: 144 large tiles
    // x 4 slices = 2.25 rounds, 357 us; 576 small tiles x 2 slices 313 us).  Slices of 1024 K
    // values and more only: that is what the model was fitted to.
    if (kind == pgk::TILE_LARGE || kind == pgk::TILE_SMALL) {
        auto estimate = [&](int knd, int64_t n) {
            const double second_pass = 2.0 * (double)n * (double)M * (double)N * (double)batch * 4.0 / 4.0e6 + 5.0;
            return estimated_rounds_time(M, N, (K + n - 1) / n, dtype, batch * n, knd) + (n > 1 ? second_pass : 0.0);
        };
        const int other = kind == pgk::TILE_LARGE ? pgk::TILE_SMALL : pgk::TILE_LARGE;
        const long double other_target = (dtype == PGK_DTYPE_F32 && other == pgk::TILE_SMALL   ? 4.0L
                                          : dtype == PGK_DTYPE_BF16 && other == pgk::TILE_LARGE ? 1.0L
                                                                                                 : 2.0L) * kNumCUs;
        const int64_t s_other = slices_for(tiles_of(other), other_target);
        // (A large tile that fits in one round is better than the model has it.  bf16: 8 x [256 x 384 x 64992] on small
        // tiles, estimated at 0.89 of it, 184 us, on large ones 167.  fp32, whose fit is that of the fp32 instruction: the factor
        // of auto_tile_kind; 9 x [256 x 130 x 53517] 409 and 366, 16 x [128 x 192 x 24994] 194 and 173.)
        const bool one_round = fit_round && kind == pgk::TILE_LARGE && tiles * s <= target;
        const double margin = !one_round ? 0.94 : dtype == PGK_DTYPE_BF16 ? 0.88 : 0.78;
        const bool other_allowed = other == pgk::TILE_SMALL || !large_tile_mostly_empty(M, N, dtype);
        if (other_allowed && K / s >= 1024 && K / s_other >= 1024 && estimate(other, s_other) < margin * estimate(kind, s)) {
            kind = other;
            s = s_other;
        }
    }
    return {(int)s, kind};
}

// Slices and large tiles that fit one round are faster (fp32 8 x [256 x 384 x 64992], 6 slices of small tiles or 10 of large ones, 923 / 646 us,
// bf16 10 x [512 x 500 x 20000], 4 or 6, 200 / 135), and taken where no sum gets less exact by them: with no fewer slices, whose
// chains of sums would be longer (512 x 178 x 19776, 13 entries, error 1.33e-6 in four slices, 1.55e-6 in three), and not from the fp32 large tile,
// which computes in bf16 terms, to the small one, whose sums are those of the fp32 instruction (320 x 157 x 8029, 11 entries, 1.7e-7 and 6.7e-7).
AutoPlan auto_split(int64_t M, int64_t N, int64_t K, int64_t batch, int dtype)
{
    const AutoPlan plain = count_slices(M, N, K, batch, dtype, false), fitted = count_slices(M, N, K, batch, dtype, true);
    const bool rounder = dtype == PGK_DTYPE_F32 && plain.kind == pgk::TILE_LARGE && fitted.kind != pgk::TILE_LARGE;
    return fitted.splits >= plain.splits && !rounder ? fitted : plain;
}

SplitPlan plan_splits(int64_t M, int64_t N, int64_t K, int64_t batch, int dtype, int splits)
{
    const int ks = kstep_of(dtype);
    const int64_t ksteps = (K + ks - 1) / ks;
    int64_t s = splits;
    if (s == 0) {
        if (mfma_route(M, N, K, dtype)) {
            s = auto_split(M, N, K, batch, dtype).splits;
        } else {
            const pgk::TileShape t = pgk::guarded_tile_shape();
            const long double tiles = (long double)((M + t.bm - 1) / t.bm) * ((N + t.bn - 1) / t.bn) * batch;
            s = 1;
            while (s < kMaxAutoSplits && s < ksteps && tiles * s < 2.0L * kNumCUs) ++s;
        }
    }
    if (s > ksteps) s = ksteps;
    const int64_t per = (ksteps + s - 1) / s;     // K steps per slice
    const int64_t L = per * ks;
    const int64_t eff = (K + L - 1) / L;          // drop trailing empty slices
    return {(int)eff, (int)L};
}

// an automatic plan comes with its tile; explicit splits get the tile their grid suggests (-1)
int split_tile_kind(int64_t M, int64_t N, int64_t K, int64_t batch, int dtype, int splits)
{
    return (splits == 0 && mfma_route(M, N, K, dtype)) ? auto_split(M, N, K, batch, dtype).kind : -1;
}

int group_m_for(int tiles_m, int tiles_n)
{
    // 32 workgroups of an XCD run together; keep their tiles near-square.
    int g = tiles_n >= 8 ? 4 : 8;
    if (g > tiles_m) g = tiles_m;
    return g;
}

struct Path { bool mfma; int kind; pgk::TileShape tile; };

// Half of a large tile (tall: half as wide; wide: half as high) when that takes away at least
// a third of the padded area the large tiles would compute -- the last tile column or row at
// most half full and few of them -- and still gives a grid that fills the chip.  (With less
// padding to save the large tile's better main loop wins: a half tile moves three quarters of
// the operand bytes per K tile for half the matrix work.)
int half_tile_kind(int64_t M, int64_t N, int dtype, int64_t units, bool b_trans)
{
    const pgk::TileShape big = pgk::mfma_tile_shape(dtype, pgk::TILE_LARGE);
    const long double area_large = (long double)((M + big.bm - 1) / big.bm * big.bm) * ((N + big.bn - 1) / big.bn * big.bn);
    for (int kind : {pgk::TILE_TALL, pgk::TILE_WIDE}) {
        if (!pgk::mfma_has_tile(dtype, kind, b_trans)) continue;
        const pgk::TileShape t = pgk::mfma_tile_shape(dtype, kind);
        const int64_t tm = (M + t.bm - 1) / t.bm, tn = (N + t.bn - 1) / t.bn;
        const long double area = (long double)(tm * t.bm) * (tn * t.bn);
        if (3 * area <= 2 * area_large && (long double)tm * tn * units >= 0.75L * kNumCUs) return kind;
    }
    return -1;
}

// The tile shape for an output of M x N with `units` workgroups per tile position (batch entries
// x K splits): the small tile when three quarters of a large tile would be empty, else a half
// tile when that saves a third of the padding, else the small tile when the large-tile grid would
// leave a quarter of the CUs idle or K is at most two bf16 K tiles, else the large tile -- unless its grid ends in a poorly
// filled round and the round model above gives another shape at least 6 % less time (K below
// 1024: the model is not consulted).
// Latency-bound fp32 problems: so few 64 x 64 tiles that most of the chip would idle behind one
// chain of K/2 dependent matrix instructions per wave, and a K too short for a two-pass split.
// They run on 32 x 32 tiles whose four waves split the K range (256 x 256 x 256: 16 workgroups
// with chains of 128 instructions become 64 workgroups with chains of 32).
bool tiny_problem(int64_t M, int64_t N, int64_t K, int dtype, int64_t units, bool b_trans, int64_t ldb)
{
    if (dtype != PGK_DTYPE_F32 || b_trans || K < 64 || K % 4 || N % 4 || (ldb ? ldb : N) % 4) return false;
    if (M <= 32 || N <= 32) return false;                       // (the skinny tiles' business)
    const long double tiles64 = (long double)((M + 63) / 64) * ((N + 63) / 64) * units;
    const int64_t ksteps = (K + 31) / 32;
    return tiles64 <= 64.0L && ksteps < 2 * 16;                 // (from 2 x 16 K tiles on, the K range is split in two passes)
}

int auto_tile_kind(int64_t M, int64_t N, int64_t K, int dtype, int64_t units, bool b_trans, int64_t ldb = 0)
{
    // (K = 0: a convolution, which keeps to the shapes its operand views were written for)
    if (const int skinny = skinny_tile_kind(M, N); K > 0 && skinny >= 0 && pgk::mfma_has_tile(dtype, skinny, b_trans)) return skinny;
    if (K > 0 && tiny_problem(M, N, K, dtype, units, b_trans, ldb)) return pgk::TILE_TINY;
    if (large_tile_mostly_empty(M, N, dtype)) return pgk::TILE_SMALL;
    if (const int half = half_tile_kind(M, N, dtype, units, b_trans); half >= 0) return half;
    // One or two bf16 K tiles: there is no main loop for the large tile to be good at, and two small
    // workgroups per CU overlap one's copies and stores with the other's (8192 x 8192 x 64 46 -> 39 us,
    // 96 x [1024 x 1024 x 64] 58 -> 52 us).  Not with output rows of 32 KiB and more, where the 256-byte
    // pieces of a small tile's rows lie too far apart for the memory (16384 x 16384 x 128: 158 against 171 us).
    if (dtype == PGK_DTYPE_BF16 && K > 0 && K <= 128 && N < 16384) return pgk::TILE_SMALL;
    const pgk::TileShape big = pgk::mfma_tile_shape(dtype, false);
    const long double wgs = (long double)((M + big.bm - 1) / big.bm) * ((N + big.bn - 1) / big.bn) * units;
    if (dtype == PGK_DTYPE_BF16) {
        // One large tile fits a CU, two small ones, one half tile.  Up to half the CUs' worth of
        // large tiles the half and small tiles still run in a single round and win (2560 x 3072 x
        // 4096, 120 large tiles: 75 us large, 62 small, 55 tall); one large tile more and they
        // need a second round while the large tiles do not (2816 x 3072 x 4096, 132: 78 us large,
        // 86 small, 100 tall; the same up to 196).  With at least 192 of them the tall tile is
        // the better single round from 16 K tiles on (5-12 % ahead of the small one).
        if (wgs <= 0.5L * kNumCUs)
            return (K >= 1024 && 2 * wgs >= 0.75L * kNumCUs && pgk::mfma_has_tile(dtype, pgk::TILE_TALL, b_trans)) ? pgk::TILE_TALL
                                                                                                                : pgk::TILE_SMALL;
    } else if (wgs < 0.75L * kNumCUs) {
        return pgk::TILE_SMALL;
    }
    int best = pgk::TILE_LARGE;
    if (K >= 1024 && wgs > kNumCUs) {      // (the fit does not hold for short K, where the epilogues weigh more)
        double best_time = 0.94 * estimated_rounds_time(M, N, K, dtype, units, pgk::TILE_LARGE);
        // The fp32 constants (tile_cost) were fitted when both fp32 tiles used the fp32 matrix instruction.  On
        // the bf16 matrix cores the large tile takes 0.77 of that (4096 x 4096 x 4096, four rounds: 916 us, now
        // 700), which moves the line between the tiles wherever the last round does its share of work: shapes
        // of 130 ... 6000 rows and columns (and 130 x 15000 ... 40000), K of 1024 ... 4096, batches up to 25, with a last round
        // over a quarter of the CUs.  The factor is where both tiles take the same time: of the 791 shapes that 0.75
        // gives to the large tile and 0.78 to the small one the ratio of their times has the median 0.995
        // (0.89 ... 1.10), from 0.78 to 0.82 the large tile is 1.03 times as fast; over all that it is chosen for,
        // 1.2 (0.94 for single shapes of 130 rows).  With a shorter last round it is anything
        // from 0.94 to 1.40, and the former line stands.  The slice
        // counts of automatic splits, and with them the workspace a call needs, stay at the former fit.
        const long double last_round = std::fmod(wgs, (long double)kNumCUs);
        if (dtype == PGK_DTYPE_F32 && (last_round == 0 || last_round > 0.25L * kNumCUs)) best_time *= 0.78;
        for (int kind : {pgk::TILE_SMALL, pgk::TILE_TALL, pgk::TILE_WIDE}) {
            if (!pgk::mfma_has_tile(dtype, kind, b_trans)) continue;
            const double t = estimated_rounds_time(M, N, K, dtype, units, kind);
            if (t < best_time) { best_time = t; best = kind; }
        }
    }
    return best;
}

// The tile of operands copied through registers: the large one where it is planned and has an instance (one operand of a
// plain B), else the small one, whose two workgroups per CU cover one's loads and LDS writes with the other's products.
// (The half tiles, both operands through registers, one workgroup per CU, over 73 shapes: 0.92 and 0.94 of its speed; the
// tall one 1344 x 87 x 708, 43 entries, 57 us, the small one 34, but 171 x 32134 x 6733 192 and 207.)  Slices that are planned for large tiles stay as they are: fewer would be
// longer chains of sums; whether such a grid pays is reg_copies_pay's business.
int reg_tile_kind(int kind, OddRows odd, bool b_trans)
{
    return kind == pgk::TILE_LARGE && !b_trans && !(odd.a && odd.b) ? pgk::TILE_LARGE : pgk::TILE_SMALL;
}

// kind_forced: -1 = auto_tile_kind, else the caller (an automatic split plan, a convolution plan) decides.
// `aligned`: A, B and the split-K partial products start on 16-byte boundaries (C, the biases and
// the row sums only need the alignment of their elements: a row of C may start anywhere, so its
// 16-byte stores are element-aligned ones in any case).
Path choose_path(bool aligned, int64_t M, int64_t N, int64_t K, int dtype, int64_t units, int kind_forced = -1,
                 bool b_trans = false, int64_t ldb = 0)
{
    const bool ok = aligned && mfma_shape_ok(M, N, K, dtype, b_trans, ldb);
    if (!ok) return Path{false, false, pgk::guarded_tile_shape()};
    int kind = kind_forced >= 0 ? kind_forced : auto_tile_kind(M, N, K, dtype, units, b_trans, ldb);
    if (!pgk::mfma_has_tile(dtype, kind, b_trans)) kind = pgk::TILE_SMALL;      // (the narrow tile with a plain B)
    if (const OddRows odd = odd_rows(K, dtype, b_trans, ldb ? ldb : N); odd.a || odd.b) kind = reg_tile_kind(kind, odd, b_trans);
    return Path{true, kind, pgk::mfma_tile_shape(dtype, kind)};
}

// rows of B (of Bt) `ldb` elements apart instead of N (of K)
void set_ldb(GemmArgs& a, int64_t ldb)
{
    a.ldb = (int)ldb;
    a.b_batch_stride = (long long)(a.b_trans ? a.N : a.K) * ldb;
}

// call when the views are final: rows off 4-byte boundaries, rows of a plain B that are not whole chunks
void mark_ragged_rows(GemmArgs& a, int dtype)
{
    const OddRows odd = odd_rows(a.K, dtype, a.b_trans != 0, a.ldb);
    a.reg_a = odd.a ? 1 : 0;
    a.reg_b = odd.b ? 1 : 0;
    a.b_tail_bounded = (!a.b_trans && a.ldb % chunk_elems(dtype) != 0) ? 1 : 0;
}

// One tile column (or, with a transposed B, one tile row): the workgroups stream disjoint rows of
// the large operand, K along the rows, and share only the small one.  Their K loops then start
// at different tiles, so that power-of-two row strides do not send every workgroup to the same
// memory channels at once.  With several batch entries the starting tile goes by entry: the
// workgroups of one entry share its small operand and walk K together (rotated against each
// other they fetched it several times: 32 x [2048 x 128 x 2048] bf16 47 -> 53 us).  Not when a single
// entry's shared operand is too large to stay in L2 (walking K in step, they fetch each of its
// tiles once), not with several tile columns and rows (they
// share panels of both operands), and not for a tile row over a plain B, which reads whole rows
// of B side by side with its neighbours -- the pattern the memory likes best (16 x 16384 x 16384
// fp32: 183 us, rotated 214 us).  Whole K tiles only: a partial tile has to come last.
void mark_k_rotation(GemmArgs& a, int dtype, const pgk::TileShape& t)
{
    const long double es = dtype == PGK_DTYPE_BF16 ? 2 : 4, small = 2.0e6L;
    // (with several batch entries the rotation goes by entry and the tiles of one entry stay in
    // step, so the size of what they share does not matter)
    const bool streams_a = a.tiles_n == 1 && a.tiles_m > 1 && (a.batch > 1 || (long double)a.K * a.N * es <= small);
    const bool streams_bt = a.tiles_m == 1 && a.tiles_n > 1 && a.b_trans && (a.batch > 1 || (long double)a.K * a.M * es <= small);
    a.k_rotate = ((streams_a || streams_bt) && a.K % t.bk == 0 && a.k_slice % t.bk == 0 && !a.b_tail_bounded) ? 1 : 0;
}

// The two passes of the split-K path.  `workspace`: batch * plan.splits * M * N floats;
// `part`: batch * nseg * M floats when rowsum != nullptr and the second pass uses nseg > 1
// column segments (nseg from splitk_reduce_segments), else unused.  A, B and the workspace
// start on 16-byte boundaries.
int run_split_passes(const void* A, const void* B, const float* bias, void* C, float* rowsum, int64_t M, int64_t N,
                     int64_t K, int64_t batch, int act, int dtype, const SplitPlan& plan, int small_tile,
                     float* workspace, float* part, hipStream_t st, bool aligned, bool b_trans, int64_t ldb = 0)
{
    Path path = choose_path(aligned, M, N, K, dtype, batch * plan.splits, small_tile, b_trans, ldb);
    // (the K-splitting tile of latency-bound problems has no first-pass form: its slices are its waves)
    if (path.mfma && path.kind == pgk::TILE_TINY)
        path = choose_path(aligned, M, N, K, dtype, batch * plan.splits, pgk::TILE_SMALL, b_trans, ldb);
    const int64_t tiles_m = (M + path.tile.bm - 1) / path.tile.bm;
    const int64_t tiles_n = (N + path.tile.bn - 1) / path.tile.bn;
    if ((long double)tiles_m * tiles_n * batch * plan.splits > 2.0e9L) return PGK_ERR_UNSUPPORTED;

    GemmArgs a{};
    a.A = A; a.B = B; a.bias = nullptr; a.C = nullptr; a.rs_part = nullptr;
    a.ws = workspace;
    a.M = (int)M; a.N = (int)N; a.K = (int)K; a.batch = (int)batch;
    pgk::fill_plain_views(a);
    if (b_trans) pgk::set_b_transposed(a);
    if (ldb) set_ldb(a, ldb);
    mark_ragged_rows(a, dtype);
    a.act = PGK_ACT_NONE; a.splits = plan.splits; a.k_slice = plan.k_slice;
    a.tiles_m = (int)tiles_m; a.tiles_n = (int)tiles_n;
    a.group_m = group_m_for(a.tiles_m, a.tiles_n);

    if (path.mfma) mark_k_rotation(a, dtype, path.tile);
    hipError_t e = path.mfma ? pgk::launch_gemm_mfma(a, dtype, path.kind, 1, st) : pgk::launch_gemm_guarded(a, dtype, 1, st);
    if (e != hipSuccess) return PGK_ERR_HIP;
    const int nseg = pgk::splitk_reduce_segments((int)M, (int)N, (int)batch);
    float* rs_part = (rowsum && nseg > 1) ? part : nullptr;
    e = pgk::launch_splitk_reduce(a.ws, bias, C, rowsum, rs_part, nseg, (int)M, (int)N, (int)batch, plan.splits, act, dtype, st);
    if (e != hipSuccess) return PGK_ERR_HIP;
    if (rs_part) e = pgk::launch_rowsum_combine(rs_part, rowsum, (int)M, (int)batch, nseg, st);
    return e == hipSuccess ? PGK_OK : PGK_ERR_HIP;
}

size_t split_part_bytes(int64_t M, int64_t N, int64_t batch, bool rowsum)
{
    const int nseg = pgk::splitk_reduce_segments((int)M, (int)N, (int)batch);
    return (rowsum && nseg > 1) ? (size_t)batch * (size_t)nseg * (size_t)M * sizeof(float) : 0;
}

// Products of few rows whose workgroups take all of K, in one launch (pgk_gemm_stream.hip): where that beat the skinny
// tiles with their K slices and second launch over 800 shapes of 1 ... 32 rows, 256 ... 32768 columns, K of 64 ... 16384, up to 450 entries (whole
// calls in a graph, operands from memory; tiles / one launch).  `tiles`: the workgroups that the tiles have before K is split.
// Many of them fill the chip by themselves, and the narrow workgroups of a transposed B then cost more than they spare.
//  * B transposed, up to 16 rows.  8 x 11008 x 4096 bf16 19.7 / 17.5 us, fp32 41.5 / 35.2, 1 x 4096 x 4096 13.9 / 7.4.  The limits of `tiles`: fp32
//    3 x 1053 x 1536 23 / 14 at 63, 6 x 2240 x 2042 27 / 20 at 216, 11 x 1152 x 1200 34 / 37 at 288, 4 x 4669 x 726 30 / 19 at 111, 10 x 640 x 320 27 / 48 at 695,
//    11 x 1664 x 192 8.1 / 7.3 at 91, 13 x 4688 x 127 8 / 13 at 111; bf16 12 x 6784 x 1024 18 / 14 at 159, 13 x 4405 x 1280 28 / 31 at 315, 3 x 5201 x 896 11 / 8 at 82, 12
//    x 4672 x 650 12.5 / 14.7 at 148, 2 x 960 x 448 7.9 / 6.9 at 48, 6 x 704 x 448 8 / 12 at 84, 12 x 8064 x 320 38 / 211 at 2898; with odd rows 12 x 2449 x 811 32 / 22 at
//    180, 8 x 3810 x 545 56 / 59 at 630, 5 x 1920 x 121 9.6 / 6.0 at 45, 10 x 1313 x 89 12.5 / 15.6 at 165.  Short rows of bf16 are too little for a step of 128:
//    10 x 3008 x 192 4.9 / 5.6.  A long K needs many columns (10 x 896 x 7667 21 / 25); fp32 beyond 4096 is even at best (5312 x 11136
//    51 / 67), as are wide ones (15 x 12506 x 3431 48 / 59).
//  * B plain, bf16, up to 16 rows.  8 x 11008 x 4096 19.7 / 18.4, 9 x 13248 x 2624 25 / 17, 13 x 2616 x 832, 5 entries, 11.7 / 10.1; longer K loses (7 x
//    5120 x 7808 27 / 43), many tiles are even (4 x 2176 x 344, 36 entries, 15.5 / 13.9; 2 x 6768 x 1308, 7 entries, 30 / 38).
//  * ... with odd rows, up to 32 rows: it spares the padded copy of B as well.  23 x 12131 x 5554 70 / 43, 10 x 1728 x 221, 63 entries,
//    37 / 16; few columns under a long K lose (32 x 3072 x 4429 31 / 39, 26 x 4509 x 8104 53 / 59; 9 x 8027 x 12583 110 / 81).
//  * B plain, fp32, up to 16 rows.  12 x 5376 x 1024 8.8 / 6.4, 6 x 2176 x 295, 3 entries, 11 / 5.6; 1 x 3072 x 958, 12 entries, 41 / 38 at 288, 7 x 2281 x 448,
//    70 entries, 60 / 82; K beyond 1024: 9 x 10752 x 2179 29 / 24, 8 x 25481 x 1600 41 / 42; beyond 2048: rows on 64 bytes and 10240 ... 16384
//    columns (8 x 11008 x 4096 40.3 / 32.7, 14 x 13248 x 4224 54 / 44; 15 x 12933 x 4352 48 / 57, 9 x 5228 x 4672 29 / 43, 13 x 18048 x 2210 40 / 47).
// Beyond a K of 8192 only odd rows gain (bf16, B transposed, 6 x 14592 x 8704 55 / 59; fp32 9 x 12544 x 10368 94 / 105). A second
// row block (17 ... 32 rows) loses but for odd rows.
//
// no_copies: odd rows whose operands would be copied first, for a workspace without room for that: whatever the kernel takes.
bool stream_plan(int64_t M, int64_t N, int64_t K, int64_t batch, int dtype, bool b_trans, pgk::StreamPlan* pl, bool no_copies = false)
{
    const bool f32 = dtype == PGK_DTYPE_F32;
    const bool odd = !f32 && (K % 2 != 0 || (!b_trans && N % 2 != 0));
    if (M > 32 || K < 64 || K > (odd ? 16384 : 8192) || N < 256) return false;
    if (M > 16 && (b_trans || !odd)) return false;
    const int64_t tiles = (N + 127) / 128 * batch;
    const bool any = no_copies && odd;
    if (b_trans && any) {
        pl->blocks = 1;
    } else if (b_trans) {
        if (!f32 && !odd && K < 256) return false;
        const int64_t most = odd ? (K >= 512 ? 192 : 128) : f32 ? (K >= 1024 ? 192 : K >= 256 ? 128 : 64) : K >= 1024 ? 160 : K >= 512 ? 96 : 48;
        if (tiles > most || N > 16384 || (K < 1024 && N > 8192)) return false;
        if (K > 2048 && N < (odd ? 2048 : 4096)) return false;
        if (f32 && (K > 4096 || (K > 2048 && N > 12288))) return false;
        pl->blocks = 1;
    } else if (!f32) {
        if (any ? false : odd ? K > 4096 && (N < 4096 || 5 * N < 3 * K) : tiles >= 128 || K > 4096 || (N <= 4096 && K > 1024)) return false;
        pl->blocks = N >= 16384 && K <= 8192 ? 8 : 4;   // (8 / 4: 24 x 16387 x 4095 58 / 78 us, 16 x 11008 x 4095 38 / 31; 15001 x 2048 19 / 21)
    } else {
        if (tiles > 320 || N > 32768 || (K > 1024 && (N <= 4096 || N > 16384))) return false;
        if (K > 2048 && (N < 10240 || N % 16 != 0)) return false;
        pl->blocks = N >= 4096 ? 4 : 2;
    }
    // A wave's sum runs over K / waves products, and the error grows with the length of that chain (fp32 8 x 4096 x 8192 4.2e-7
    // in 16 slices, 5.8e-7 in eight waves).  The tiles' slices are 16 K tiles or longer, 512 products of fp32 and 1024 of bf16, and from
    // 10240 columns on at most seven of them; the waves' chains are at most 512 of fp32 up to a K of 4096 and 1024 above, and 1024 of
    // bf16.  (Sixteen waves for a longer K, fp32, B transposed, 5312 x 5851: 45 us, eight 41, in slices 37.)
    pl->waves = K > 8192 ? 16 : b_trans || K > 1024 ? 8 : 4;
    const int64_t cols = 16 * pl->blocks, groups = (N + cols - 1) / cols;
    pl->groups = (int)std::min<int64_t>(groups, kMaxDim);
    return pgk::stream_launch_fits(*pl, batch);
}

// What pgk_gemm_fused does with a problem: the kernel and tile of the single-pass route, and
// whether the K range is split instead (then `slices` and the tile that goes with them).
struct FusedPlan {
    Path path;
    bool split;
    SplitPlan slices;
    int split_small_tile;
};

FusedPlan plan_fused(bool aligned, int64_t M, int64_t N, int64_t K, int64_t batch, int dtype, bool b_trans, int64_t ldb = 0)
{
    FusedPlan fp{};
    fp.path = choose_path(aligned, M, N, K, dtype, batch, -1, b_trans, ldb);
    const int64_t tiles_m = (M + fp.path.tile.bm - 1) / fp.path.tile.bm;
    const int64_t tiles_n = (N + fp.path.tile.bn - 1) / fp.path.tile.bn;
    // Few output tiles and a long K (skinny or small outputs): one workgroup per tile would
    // leave most of the chip idle, so the K range is split as in pgk_gemm_splitk, with the
    // partial products in the caller's workspace.  The choice depends on the shape only.
    // (Also when only the small-tile grid fills the chip and K is very long: 256 x 256 x 65536 x 16
    // fp32 took 1536 us on 256 small tiles and 1083 us split; below 512 K tiles the split's extra
    // pass costs more than it gains -- 2048 x 2048 x 16384 bf16: 130 us against 152 us.)
    const pgk::TileShape big = pgk::mfma_tile_shape(dtype, false);
    const long double big_tiles = (long double)((M + big.bm - 1) / big.bm) * ((N + big.bn - 1) / big.bn) * batch;
    // (skinny tiles run at the speed of their operand stream, which takes two workgroups per CU
    // to keep busy: 16 x 32000 x 4096 fp32, 250 flat tiles, 122 us in one piece and 94 us in two slices)
    const bool skinny = fp.path.kind == pgk::TILE_NARROW || fp.path.kind == pgk::TILE_FLAT;
    // (a bf16 large-tile grid is only chosen from half the CUs' worth of tiles on, and then runs
    // in one piece: two slices of 160 tiles would be a round and a quarter plus the second pass)
    const bool bf16_large = dtype == PGK_DTYPE_BF16 && fp.path.kind == pgk::TILE_LARGE;
    const bool few_tiles = !bf16_large &&
                           (long double)tiles_m * tiles_n * batch < (skinny ? (3 * kNumCUs) / 2 : (3 * kNumCUs) / 4);
    const bool long_k = !bf16_large && big_tiles < (3 * kNumCUs) / 4 && (K + big.bk - 1) / big.bk >= kLongKSteps;
    // (The fp32 small tile fits a CU four times; a grid that fills less than three quarters of
    // those places leaves each CU with one wave per SIMD and nothing to hide its waits behind.
    // From 128 K tiles on the split pays: 16384 x 64 x 8192 275 -> 173 us, 1024 x 1024 x 4096 81 -> 72 us;
    // at 64 K tiles it is even, at 32 it loses.)
    const bool under_filled = dtype == PGK_DTYPE_F32 && fp.path.kind == pgk::TILE_SMALL &&
                              (long double)tiles_m * tiles_n * batch < 3 * kNumCUs && (K + big.bk - 1) / big.bk >= 128;
    if (fp.path.mfma && (few_tiles || long_k || under_filled)) {
        fp.slices = plan_splits(M, N, K, batch, dtype, 0);
        fp.split_small_tile = auto_split(M, N, K, batch, dtype).kind;
        const long double ws_bytes = (long double)batch * fp.slices.splits * M * N * sizeof(float);
        fp.split = fp.slices.splits > 1 && ws_bytes <= (long double)kAutoSplitMaxWorkspace;
    }
    return fp;
}

// K tiles of a workgroup (one slice): those of the main loop, and those at its end that are loaded with waits and run-time
// checks (the loop goes in trips of six, or of two; the last two load nothing any more).  whole: the last K tile is no edge.
struct LoopTiles { double steady, tail; };

LoopTiles loop_tiles(int64_t K, int count, bool whole, int trip)
{
    const int64_t n = ((K + 63) / 64 + count - 1) / count, m = n - (whole ? 0 : 1);
    const int64_t rest = n - (m > trip + 1 ? (m - 2) / trip * trip : 0);
    return {(double)(n - std::max<int64_t>(rest - 2, 0)), (double)std::max<int64_t>(rest - 2, 0)};
}

// Whether operands with odd rows are copied through registers (pgk_gemm_mfma_reg.hip) or first into rows padded to whole
// chunks (pack_dims): both ways as they would be planned, in microseconds on the measured part.  A round of workgroups takes a
// fixed time and so much per K tile, more for those at a loop's end, and a last round with one workgroup on its busiest CU a time of its own.  K tiles
// through registers take 1.25 to 1.5 times as long, and 1.1 times that with A so on the large tile, with both operands odd or B
// transposed on the small one; the copies read and write at 5 TB/s, an odd K both operands, rows of a plain B it alone, and take 2.4 us a launch.
// Output rows off the 16-byte grid take 0.14 us a megabyte more, 0.03 with the plain stores of the register instances.
// Fitted to 6400 fused calls (33 ... 16384 x 33 ... 50257 x 33 ... 16384, batches up to 64, both layouts of B, up to 1.5 TFLOP).  On 2000 others: 0.6 %
// above the better of both ways in the geometric mean (copies always 16 %, registers always 5 %), 50 of the choices more than 5 % slower
// than the copies, 50 than the registers; 600 split calls 1.2 %.
// Copied first / through registers: 512 x 50257 x 768 83 / 70 us, 128 x 256 x 32371, 16 entries, 228 / 96, 9800 x 12713 x 64
// 139 / 89, 1024 x 2048 x 255 (B transposed) 14 / 11; 2048 x 2047 x 2048 34 / 46, 4096 x 4095 x 4095 132 / 213, 16 x [1501 x 1501 x 1501] 182 / 237,
// 832 x 1440 x 379 (B transposed), 32 entries, 78 / 120, 960 x 3433 x 257, 16 entries, 99 / 120.
// The fit is of main loops in trips of six; all but the large tile's with A through registers now go in trips of two, which spares some of the tiles at their
// end.  From seven K tiles on that is counted, with a margin for what has not been fitted: 70 drawn products whose choice it turns to registers
// are 1.05 to 1.44 times as fast, 1.20 in the mean (435 x 37339 x 429, B transposed, 73 copied, 56 through registers; 7616 x 53 x 1225 37 and 26).
bool reg_copies_pay(int64_t M, int64_t N, int64_t K, int64_t batch, int dtype, bool b_trans, Slices slices)
{
    // a round: fixed + steady and tail K tiles; the last one: with one workgroup on its busiest CU, and with two, as a share
    struct Cost { double fixed, steady, tail, lone_fixed, lone_steady, lone_tail, two; };
    auto time = [](const Cost& c, LoopTiles t, Rounds r, double loop) {
        const double round = c.fixed + loop * (c.steady * t.steady + c.tail * t.tail);
        const double lone = c.lone_fixed + loop * (c.lone_steady * t.steady + c.lone_tail * t.tail);
        return round * (r.full + (r.rest > 1 ? c.two : 0.0)) + (r.rest == 1 ? lone : 0.0);
    };
    auto packed_cost = [](int kind) -> Cost {
        switch (kind) {
        case pgk::TILE_LARGE: return {5.5, 1.24, 1.86, 6.4, 1.07, 2.21, 1.0};
        case pgk::TILE_TALL: return {5.3, 0.95, 1.51, 4.1, 0.74, 1.18, 1.0};
        case pgk::TILE_WIDE: return {3.3, 0.84, 1.33, 3.5, 0.88, 1.41, 1.0};
        default: return {3.0, 0.85, 2.02, 1.8, 0.52, 1.24, 0.84};
        }
    };
    auto reg_cost = [](int kind) -> Cost {
        if (kind == pgk::TILE_LARGE) return {4.6, 1.53, 2.43, 4.5, 1.45, 2.16, 1.0};
        return {2.5, 1.23, 2.30, 2.1, 0.78, 1.84, 0.93};
    };
    struct Planned { int kind, count; Rounds rounds; };
    auto plan = [&](int64_t k, int64_t ldb) {
        Planned p{slices.kind, slices.count, {}};
        if (!p.count) {
            const FusedPlan fp = plan_fused(true, M, N, k, batch, dtype, b_trans, ldb);
            p.count = fp.split ? fp.slices.splits : 1;
            p.kind = fp.split ? fp.split_small_tile : fp.path.kind;
        }
        p.kind = choose_path(true, M, N, k, dtype, batch * p.count, p.kind, b_trans, ldb).kind;
        p.rounds = rounds_of(M, N, dtype, batch * p.count, p.kind);
        return p;
    };
    const OddRows odd = odd_rows(K, dtype, b_trans, N);
    const int64_t epc = chunk_elems(dtype), k = odd.a ? round_up64(K, epc) : K;
    const Planned reg = plan(K, 0), packed = plan(k, b_trans ? k : round_up64(N, epc));
    const double in = (double)K * (double)batch * 2.0e-6, out = (double)M * (double)N * (double)batch * 2.0e-6;    // MB (in: a row's)
    const double partials = 0.6 * out;                                     // (a slice's, written and read)

    const double loop = reg.kind == pgk::TILE_LARGE ? (odd.a ? 1.09 : 1.0) : b_trans ? 1.13 : odd.a && odd.b ? 1.11 : 1.0;
    auto by_reg = [&](int trip) {
        return time(reg_cost(reg.kind), loop_tiles(K, reg.count, false, trip), reg.rounds, loop) +
               in * (0.17 * (double)M + 0.14 * (double)N) + (N % 8 != 0 ? 0.17 : 0.14) * out + (reg.count > 1 ? reg.count * partials : 0.0);
    };
    const double by_copies = time(packed_cost(packed.kind), loop_tiles(k, packed.count, k % 64 == 0, 6), packed.rounds, 1.0) +
                             in * ((odd.a ? 0.41 * (double)M : 0.0) + (b_trans ? 0.39 : 0.34) * (double)N) +
                             (odd.a ? 4.8 : 2.2) + (N % 8 != 0 ? 0.20 : 0.06) * out + (packed.count > 1 ? packed.count * partials : 0.0);
    if (by_reg(6) < by_copies) return true;
    const bool long_enough = (K + 63) / 64 >= 7 * (int64_t)reg.count;
    return long_enough && !(reg.kind == pgk::TILE_LARGE && odd.a) && by_reg(2) < 0.95 * by_copies;
}

// ---- The caller's workspace.  Everything a call needs beyond its inputs and outputs is cut from
// it, each piece starting on a multiple of 256 bytes from its (16-byte aligned) base:
//   products  split-K partial products [batch][slices][M][N] fp32 (first, at offset 0)
//   rs_part   row-sum partials, per tile column (single pass) or per column segment (second pass)
//   pack_a/b  zero-padded (or transposed) copies of operands the kernels cannot read in place
// The sizes depend on the shape, the layout of B, whether row sums are wanted and whether A / B
// start on 16-byte boundaries -- the same function answers the workspace queries and lays the
// workspace out inside the calls.
struct WsNeeds {
    bool ok;                 // sizes are representable
    bool stream;             // fused call: the kernel for few rows
    pgk::StreamPlan sp;
    PackDims d;
    bool pack_a, pack_b;
    FusedPlan fp;            // fused call only
    size_t products, rs_part, a_bytes, b_bytes;
    size_t off_rs_part, off_a, off_b, total;
};

void lay_out(WsNeeds& w)
{
    size_t at = round_up256(w.products);
    w.off_rs_part = at; at += round_up256(w.rs_part);
    w.off_a = at; at += round_up256(w.a_bytes);
    w.off_b = at; at += round_up256(w.b_bytes);
    w.total = at;
}

// the operand copies of a packed problem (see pack_dims); a_mis / b_mis: that operand does not
// start on a 16-byte boundary
bool pack_needs(WsNeeds& w, int64_t M, int64_t N, int64_t K, int64_t batch, int dtype, bool b_trans, bool a_mis, bool b_mis,
                Slices slices)
{
    const size_t es = dtype == PGK_DTYPE_BF16 ? 2 : 4;
    w.d = pack_dims(M, N, K, batch, dtype, b_trans, slices, a_mis || b_mis);
    w.pack_a = w.pack_b = false;
    w.a_bytes = w.b_bytes = 0;
    if (!w.d.pack) return true;
    w.pack_a = w.d.k != K || a_mis;
    w.pack_b = w.d.transpose_b || w.d.k != K || (!b_trans && w.d.ldb != N) || b_mis;
    const int64_t b_rows = w.d.b_trans ? N : w.d.k;
    const long double total = (long double)batch * M * w.d.k * es + (long double)batch * b_rows * w.d.ldb * es;
    if (total >= 4.0e12L) return false;
    if (w.pack_a) w.a_bytes = (size_t)batch * (size_t)M * (size_t)w.d.k * es;
    if (w.pack_b) w.b_bytes = (size_t)batch * (size_t)b_rows * (size_t)w.d.ldb * es;
    return true;
}

// How a fused call may run: the fastest way, the tiles in any case, or with no copies of operands that only their odd rows ask for
enum class Way { fastest, tiles, no_copies };

WsNeeds fused_needs(int64_t M, int64_t N, int64_t K, int64_t batch, int dtype, bool b_trans, bool want_rowsum, bool a_mis,
                    bool b_mis, Way way = Way::fastest)
{
    WsNeeds w{};
    if (way != Way::tiles && stream_plan(M, N, K, batch, dtype, b_trans, &w.sp, way == Way::no_copies)) {
        w.ok = w.stream = true;
        w.d = PackDims{false, K, 0, false, b_trans};
        w.rs_part = (want_rowsum && w.sp.groups > 1) ? (size_t)batch * (size_t)w.sp.groups * (size_t)M * sizeof(float) : 0;
        lay_out(w);
        return w;
    }
    w.ok = pack_needs(w, M, N, K, batch, dtype, b_trans, a_mis, b_mis, Slices{0, -1, way == Way::no_copies});
    if (!w.ok) return w;
    // the problem as the kernels see it
    const bool packed = w.d.pack;
    const int64_t Kc = packed ? w.d.k : K;
    w.fp = plan_fused(packed || !(a_mis || b_mis), M, N, Kc, batch, dtype, packed ? w.d.b_trans : b_trans, packed ? w.d.ldb : 0);
    if (w.fp.split) {
        w.products = (size_t)batch * (size_t)w.fp.slices.splits * (size_t)M * (size_t)N * sizeof(float);
        w.rs_part = split_part_bytes(M, N, batch, want_rowsum);
    } else {
        const int64_t tiles_n = (N + w.fp.path.tile.bn - 1) / w.fp.path.tile.bn;
        if ((long double)batch * tiles_n * M * 4.0L >= 1.8e19L) { w.ok = false; return w; }
        w.rs_part = (want_rowsum && tiles_n > 1) ? (size_t)batch * (size_t)tiles_n * (size_t)M * sizeof(float) : 0;
    }
    lay_out(w);
    return w;
}

WsNeeds splitk_needs(int64_t M, int64_t N, int64_t K, int64_t batch, int dtype, Slices slices, bool b_trans,
                     bool want_rowsum, bool a_mis, bool b_mis)
{
    WsNeeds w{};
    w.ok = pack_needs(w, M, N, K, batch, dtype, b_trans, a_mis, b_mis, slices);
    if (!w.ok) return w;
    if ((long double)batch * slices.count * M * N * sizeof(float) >= 1.8e19L) { w.ok = false; return w; }
    w.products = (size_t)batch * (size_t)slices.count * (size_t)M * (size_t)N * sizeof(float);
    w.rs_part = split_part_bytes(M, N, batch, want_rowsum);
    lay_out(w);
    return w;
}

// What calls with `workspace_bytes` do.  The kernel for few rows has row sums per 16 to 128 columns where the tiles have them
// per 128, and odd rows that are copied first may be read in place as well: a workspace with room for the slower way is enough for it.
WsNeeds fused_needs_within(size_t workspace_bytes, int64_t M, int64_t N, int64_t K, int64_t batch, int dtype, bool b_trans,
                           bool want_rowsum, bool a_mis, bool b_mis)
{
    const WsNeeds w = fused_needs(M, N, K, batch, dtype, b_trans, want_rowsum, a_mis, b_mis);
    if (!w.ok || w.total <= workspace_bytes) return w;
    for (const Way way : {Way::tiles, Way::no_copies}) {
        const WsNeeds other = fused_needs(M, N, K, batch, dtype, b_trans, want_rowsum, a_mis, b_mis, way);
        if (other.ok && other.total <= workspace_bytes) return other;
    }
    return w;
}

WsNeeds splitk_needs_within(size_t workspace_bytes, int64_t M, int64_t N, int64_t K, int64_t batch, int dtype, Slices slices, bool b_trans,
                            bool want_rowsum, bool a_mis, bool b_mis)
{
    const WsNeeds w = splitk_needs(M, N, K, batch, dtype, slices, b_trans, want_rowsum, a_mis, b_mis);
    if (!w.ok || w.total <= workspace_bytes) return w;
    slices.no_copies = true;
    const WsNeeds other = splitk_needs(M, N, K, batch, dtype, slices, b_trans, want_rowsum, a_mis, b_mis);
    return other.ok && other.total <= workspace_bytes ? other : w;
}

bool sizes_valid(int64_t M, int64_t N, int64_t K, int64_t batch, int dtype)
{
    const void* ok = reinterpret_cast<const void*>(uintptr_t{256});
    return validate_common(ok, ok, ok, M, N, K, batch, PGK_ACT_NONE, dtype) == PGK_OK;
}

// Zero-padded copies of the operands of a packed problem (see pack_dims) into the workspace
// pieces w.off_a / w.off_b: A' [batch][M][d.k] when K is ragged or A misaligned, B' [batch][d.k][d.ldb]
// (or Bt' [batch][N][d.k]) when K or its rows are ragged or B misaligned, or when a narrow plain
// B is to be transposed (d.transpose_b; `b_trans` is the layout of the B given).
struct PackedOperands { const void* A; const void* B; };

int pack_operands(const WsNeeds& w, unsigned char* base, const void* A, const void* B, int64_t M, int64_t N, int64_t K,
                  int64_t batch, int dtype, bool b_trans, hipStream_t st, PackedOperands* out)
{
    const PackDims& d = w.d;
    *out = PackedOperands{A, B};
    hipError_t e = hipSuccess;
    if (w.pack_a) {
        unsigned char* p = base + w.off_a;
        e = pgk::launch_pad_matrix(A, p, batch, (int)M, (int)K, (int)M, (int)d.k, dtype, st);
        if (e != hipSuccess) return PGK_ERR_HIP;
        out->A = p;
    }
    if (w.pack_b) {
        unsigned char* p = base + w.off_b;
        e = d.transpose_b ? pgk::launch_transpose_pad(B, p, batch, (int)K, (int)N, (int)d.ldb, dtype, st)
            : b_trans     ? pgk::launch_pad_matrix(B, p, batch, (int)N, (int)K, (int)N, (int)d.k, dtype, st)
                          : pgk::launch_pad_matrix(B, p, batch, (int)K, (int)N, (int)d.k, (int)d.ldb, dtype, st);
        if (e != hipSuccess) return PGK_ERR_HIP;
        out->B = p;
    }
    return PGK_OK;
}

int check_workspace(const WsNeeds& w, const void* workspace, size_t workspace_bytes)
{
    if (!w.ok) return PGK_ERR_UNSUPPORTED;
    if (w.total == 0) return PGK_OK;
    if (!workspace || workspace_bytes < w.total || !aligned16(workspace)) return PGK_ERR_WORKSPACE;
    return PGK_OK;
}

// ---- pgk_gemm_fused_static: the workspace of callers that cannot supply one.  A fixed array in
// the library's device image; each GPU the library runs on holds its own copy, at its own
// address, until the process ends.  Host code never uses the array's name as a pointer: the
// device address is looked up once per device and cached.
constexpr size_t kStaticScratchBytes = (size_t)4 << 20;
constexpr int kMaxDevices = 64;
std::mutex g_static_mu;
void* g_static_ptr[kMaxDevices] = {};

int static_scratch_of_current_device(void** out)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return PGK_ERR_HIP;
    std::lock_guard<std::mutex> lk(g_static_mu);
    if (!g_static_ptr[dev]) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return PGK_ERR_HIP;
        g_static_ptr[dev] = p;
    }
    *out = g_static_ptr[dev];
    return PGK_OK;
}

// pgk_gemm_fused and pgk_gemm_fused_bt (b_trans: B given as [batch][N][K])
int gemm_fused_impl(const void* A, const void* B, const float* bias, void* C, float* rowsum,
                    int64_t M, int64_t N, int64_t K, int64_t batch, int act, int dtype,
                    void* workspace, size_t workspace_bytes, void* stream, bool b_trans)
{
    int rc = validate_common(A, B, C, M, N, K, batch, act, dtype);
    if (rc != PGK_OK) return rc;
    const bool a_mis = !aligned16(A), b_mis = !aligned16(B);
    const WsNeeds w = fused_needs_within(workspace ? workspace_bytes : 0, M, N, K, batch, dtype, b_trans, rowsum != nullptr, a_mis, b_mis);
    rc = check_workspace(w, workspace, workspace_bytes);
    if (rc != PGK_OK) return rc;
    if (w.stream)
        return pgk::launch_gemm_stream(w.sp, A, B, bias, C, rowsum, w.rs_part ? static_cast<float*>(workspace) : nullptr, (int)M,
                                       (int)N, (int)K, (int)batch, act, dtype, b_trans, static_cast<hipStream_t>(stream)) == hipSuccess
                   ? PGK_OK : PGK_ERR_HIP;
    const FusedPlan& fp = w.fp;
    const Path& path = fp.path;
    const int64_t tiles_m = (M + path.tile.bm - 1) / path.tile.bm;
    const int64_t tiles_n = (N + path.tile.bn - 1) / path.tile.bn;
    if ((long double)tiles_m * tiles_n * batch > 2.0e9L) return PGK_ERR_UNSUPPORTED;
    // ---- everything below enqueues work
    hipStream_t st = static_cast<hipStream_t>(stream);
    unsigned char* base = static_cast<unsigned char*>(workspace);
    PackedOperands pk{A, B};
    int64_t ldb = 0;
    bool aligned = !(a_mis || b_mis);
    if (w.d.pack) {
        rc = pack_operands(w, base, A, B, M, N, K, batch, dtype, b_trans, st, &pk);
        if (rc != PGK_OK) return rc;
        K = w.d.k; b_trans = w.d.b_trans; ldb = w.d.ldb;
        aligned = true;
    }
    float* part = w.rs_part ? reinterpret_cast<float*>(base + w.off_rs_part) : nullptr;

    if (fp.split)
        return run_split_passes(pk.A, pk.B, bias, C, rowsum, M, N, K, batch, act, dtype, fp.slices, fp.split_small_tile,
                                reinterpret_cast<float*>(base), part, st, aligned, b_trans, ldb);

    GemmArgs a{};
    a.A = pk.A; a.B = pk.B; a.bias = bias; a.C = C; a.ws = nullptr;
    a.M = (int)M; a.N = (int)N; a.K = (int)K; a.batch = (int)batch;
    pgk::fill_plain_views(a);
    if (b_trans) pgk::set_b_transposed(a);
    if (ldb) set_ldb(a, ldb);
    mark_ragged_rows(a, dtype);
    a.act = act; a.splits = 1;
    a.k_slice = (int)(((K + path.tile.bk - 1) / path.tile.bk) * path.tile.bk);
    a.tiles_m = (int)tiles_m; a.tiles_n = (int)tiles_n;
    a.group_m = group_m_for(a.tiles_m, a.tiles_n);
    // one tile column: the kernel's row sums are final; several: per-tile-column partials, added
    // in tile-column order by a second small kernel
    if (rowsum) a.rs_part = tiles_n == 1 ? rowsum : part;
    if (path.mfma) mark_k_rotation(a, dtype, path.tile);
    hipError_t e = path.mfma ? pgk::launch_gemm_mfma(a, dtype, path.kind, 0, st) : pgk::launch_gemm_guarded(a, dtype, 0, st);
    if (e != hipSuccess) return PGK_ERR_HIP;
    if (rowsum && tiles_n > 1) {
        e = pgk::launch_rowsum_combine(part, rowsum, (int)M, (int)batch, (int)tiles_n, st);
        if (e != hipSuccess) return PGK_ERR_HIP;
    }
    return PGK_OK;
}

}  // namespace

extern "C" {

int pgk_gemm_fused(const void* A, const void* B, const float* bias, void* C, float* rowsum,
                   int64_t M, int64_t N, int64_t K, int64_t batch, int act, int dtype,
                   void* workspace, size_t workspace_bytes, void* stream)
{
    return gemm_fused_impl(A, B, bias, C, rowsum, M, N, K, batch, act, dtype, workspace, workspace_bytes, stream, false);
}

int pgk_gemm_fused_bt(const void* A, const void* Bt, const float* bias, void* C, float* rowsum,
                      int64_t M, int64_t N, int64_t K, int64_t batch, int act, int dtype,
                      void* workspace, size_t workspace_bytes, void* stream)
{
    return gemm_fused_impl(A, Bt, bias, C, rowsum, M, N, K, batch, act, dtype, workspace, workspace_bytes, stream, true);
}

int pgk_gemm_fused_static(const void* A, const void* B, const float* bias, void* C, float* rowsum,
                          int64_t M, int64_t N, int64_t K, int64_t batch, int act, int dtype, void* stream)
{
    int rc = validate_common(A, B, C, M, N, K, batch, act, dtype);
    if (rc != PGK_OK) return rc;
    // the need is known on the host: refuse before touching the device
    const WsNeeds w = fused_needs_within(kStaticScratchBytes, M, N, K, batch, dtype, false, rowsum != nullptr, !aligned16(A), !aligned16(B));
    if (!w.ok) return PGK_ERR_UNSUPPORTED;
    if (w.total > kStaticScratchBytes) return PGK_ERR_WORKSPACE;
    void* ws = nullptr;
    if (w.total) {
        rc = static_scratch_of_current_device(&ws);
        if (rc != PGK_OK) return rc;
    }
    return gemm_fused_impl(A, B, bias, C, rowsum, M, N, K, batch, act, dtype, ws, w.total ? kStaticScratchBytes : 0, stream, false);
}

size_t pgk_gemm_fused_static_max_bytes(void) { return kStaticScratchBytes; }

size_t pgk_gemm_fused_workspace_bytes(int64_t M, int64_t N, int64_t K, int64_t batch, int dtype, int flags)
{
    if (!sizes_valid(M, N, K, batch, dtype) || (flags & ~(PGK_WS_ROWSUM | PGK_WS_B_TRANSPOSED | PGK_WS_UNALIGNED))) return 0;
    const bool mis = (flags & PGK_WS_UNALIGNED) != 0;
    const WsNeeds w = fused_needs(M, N, K, batch, dtype, (flags & PGK_WS_B_TRANSPOSED) != 0, (flags & PGK_WS_ROWSUM) != 0, mis, mis);
    return w.ok ? w.total : 0;
}

int pgk_gemm_plan(int64_t M, int64_t N, int64_t K, int64_t batch, int dtype, int b_transposed, int32_t* out)
{
    if (!out) return PGK_ERR_INVALID_ARG;
    const void* ok = reinterpret_cast<const void*>(uintptr_t{256});   // stands for any 16-byte aligned pointer
    const int rc = validate_common(ok, ok, ok, M, N, K, batch, PGK_ACT_NONE, dtype);
    if (rc != PGK_OK) return rc;
    if (pgk::StreamPlan sp; stream_plan(M, N, K, batch, dtype, b_transposed != 0, &sp)) {
        // (its workgroups are narrower than a tile; the query answers with the tiles they make up)
        const pgk::TileShape t = pgk::mfma_tile_shape(dtype, pgk::TILE_FLAT);
        const long double tiles = (long double)((N + t.bn - 1) / t.bn) * batch;
        if (tiles > 2.0e9L) return PGK_ERR_UNSUPPORTED;
        out[0] = 1;
        out[1] = t.bm; out[2] = t.bn; out[3] = t.bk;
        out[4] = 1;
        out[5] = (int32_t)tiles;
        return PGK_OK;
    }
    const PackDims d = pack_dims(M, N, K, batch, dtype, b_transposed != 0, Slices{0, -1, false});      // as pgk_gemm_fused sees the problem
    K = d.k;
    const FusedPlan fp = plan_fused(true, M, N, K, batch, dtype, d.b_trans, d.ldb);
    Path path = fp.path;
    int slices = 1;
    if (fp.split) {
        slices = fp.slices.splits;
        path = choose_path(true, M, N, K, dtype, batch * slices, fp.split_small_tile, d.b_trans, d.ldb);
    }
    const long double wgs = (long double)((M + path.tile.bm - 1) / path.tile.bm) * ((N + path.tile.bn - 1) / path.tile.bn) *
                            batch * slices;
    if (wgs > 2.0e9L) return PGK_ERR_UNSUPPORTED;
    out[0] = path.mfma ? 1 : 0;
    out[1] = path.tile.bm; out[2] = path.tile.bn; out[3] = path.tile.bk;
    out[4] = slices;
    out[5] = (int32_t)wgs;
    return PGK_OK;
}

int pgk_splitk_auto_splits(int64_t M, int64_t N, int64_t K, int64_t batch, int dtype, int splits)
{
    if (M <= 0 || N <= 0 || K <= 0 || batch <= 0) return 0;
    if (dtype != PGK_DTYPE_F32 && dtype != PGK_DTYPE_BF16) return 0;
    if (M > kMaxDim || N > kMaxDim || K > kMaxDim || batch > kMaxDim) return 0;
    if (splits < 0 || splits > K) return 0;
    return plan_splits(M, N, K, batch, dtype, splits).splits;
}

size_t pgk_gemm_splitk_workspace_bytes(int64_t M, int64_t N, int64_t K, int64_t batch, int dtype, int splits, int flags)
{
    if (!sizes_valid(M, N, K, batch, dtype) || (flags & ~(PGK_WS_ROWSUM | PGK_WS_B_TRANSPOSED | PGK_WS_UNALIGNED))) return 0;
    const int s = pgk_splitk_auto_splits(M, N, K, batch, dtype, splits);
    if (s <= 0) return 0;
    const bool mis = (flags & PGK_WS_UNALIGNED) != 0;
    const WsNeeds w = splitk_needs(M, N, K, batch, dtype, Slices{s, split_tile_kind(M, N, K, batch, dtype, splits), false}, (flags & PGK_WS_B_TRANSPOSED) != 0, (flags & PGK_WS_ROWSUM) != 0, mis, mis);
    return w.ok ? w.total : 0;
}

size_t pgk_splitk_workspace_bytes(int64_t M, int64_t N, int64_t K, int64_t batch, int dtype, int splits)
{
    // enough for either layout of B, with or without row sums, operands on 16-byte boundaries
    const size_t plain = pgk_gemm_splitk_workspace_bytes(M, N, K, batch, dtype, splits, PGK_WS_ROWSUM);
    const size_t bt = pgk_gemm_splitk_workspace_bytes(M, N, K, batch, dtype, splits, PGK_WS_ROWSUM | PGK_WS_B_TRANSPOSED);
    return plain > bt ? plain : bt;
}

}  // extern "C"

namespace {

int gemm_splitk_impl(const void* A, const void* B, const float* bias, void* C, float* rowsum,
                     int64_t M, int64_t N, int64_t K, int64_t batch, int act, int dtype, int splits,
                     void* workspace, size_t workspace_bytes, void* stream, bool b_trans)
{
    int rc = validate_common(A, B, C, M, N, K, batch, act, dtype);
    if (rc != PGK_OK) return rc;
    if (splits < 0 || splits > K) return PGK_ERR_INVALID_ARG;
    const SplitPlan plan = plan_splits(M, N, K, batch, dtype, splits);
    const int tile_kind = split_tile_kind(M, N, K, batch, dtype, splits);
    const bool a_mis = !aligned16(A), b_mis = !aligned16(B);
    const WsNeeds w = splitk_needs_within(workspace ? workspace_bytes : 0, M, N, K, batch, dtype, Slices{plan.splits, tile_kind, false}, b_trans,
                                          rowsum != nullptr, a_mis, b_mis);
    if (!w.ok) return PGK_ERR_UNSUPPORTED;
    rc = check_workspace(w, workspace, workspace_bytes);
    if (rc != PGK_OK) return rc;
    // ---- everything below enqueues work
    hipStream_t st = static_cast<hipStream_t>(stream);
    unsigned char* base = static_cast<unsigned char*>(workspace);
    float* part = w.rs_part ? reinterpret_cast<float*>(base + w.off_rs_part) : nullptr;
    // (the slices are counted in K steps, which padding K to whole chunks leaves as they are)
    if (!w.d.pack)
        return run_split_passes(A, B, bias, C, rowsum, M, N, K, batch, act, dtype, plan, tile_kind,
                                reinterpret_cast<float*>(base), part, st, !(a_mis || b_mis), b_trans);
    PackedOperands pk{};
    rc = pack_operands(w, base, A, B, M, N, K, batch, dtype, b_trans, st, &pk);
    if (rc != PGK_OK) return rc;
    return run_split_passes(pk.A, pk.B, bias, C, rowsum, M, N, w.d.k, batch, act, dtype, plan, tile_kind,
                            reinterpret_cast<float*>(base), part, st, true, w.d.b_trans, w.d.ldb);
}

}  // namespace

extern "C" {

int pgk_gemm_splitk(const void* A, const void* B, const float* bias, void* C, float* rowsum,
                    int64_t M, int64_t N, int64_t K, int64_t batch, int act, int dtype, int splits,
                    void* workspace, size_t workspace_bytes, void* stream)
{
    return gemm_splitk_impl(A, B, bias, C, rowsum, M, N, K, batch, act, dtype, splits, workspace, workspace_bytes,
                            stream, false);
}

int pgk_gemm_splitk_bt(const void* A, const void* Bt, const float* bias, void* C, float* rowsum,
                       int64_t M, int64_t N, int64_t K, int64_t batch, int act, int dtype, int splits,
                       void* workspace, size_t workspace_bytes, void* stream)
{
    return gemm_splitk_impl(A, Bt, bias, C, rowsum, M, N, K, batch, act, dtype, splits, workspace, workspace_bytes,
                            stream, true);
}

size_t pgk_reduce_max_workspace_bytes(int64_t outer, int64_t red, int64_t inner, int dtype)
{
    if (outer <= 0 || red <= 0 || inner <= 0 || (dtype != PGK_DTYPE_F32 && dtype != PGK_DTYPE_BF16)) return 0;
    if (red > (1LL << 31) - 1024) return 0;
    if ((long double)outer * (long double)inner >= 4.6e18L ||
        (long double)outer * (long double)inner * (long double)red >= 4.6e18L) return 0;
    // (the plan depends on whether X starts on a 16-byte boundary: enough for either case)
    const size_t a = pgk::plan_reduce_max(outer, red, inner, dtype, true).partial_elems;
    const size_t b = pgk::plan_reduce_max(outer, red, inner, dtype, false).partial_elems;
    return (a > b ? a : b) * 8;
}

int pgk_reduce_max(const void* X, void* out, int32_t* idx, int64_t outer, int64_t red, int64_t inner,
                   int dtype, void* workspace, size_t workspace_bytes, void* stream)
{
    if (!X || !out || outer <= 0 || red <= 0 || inner <= 0) return PGK_ERR_INVALID_ARG;
    if (dtype != PGK_DTYPE_F32 && dtype != PGK_DTYPE_BF16) return PGK_ERR_INVALID_ARG;
    if (red > (1LL << 31) - 1024) return PGK_ERR_UNSUPPORTED;
    if ((long double)outer * (long double)inner >= 4.6e18L ||
        (long double)outer * (long double)inner * (long double)red >= 4.6e18L) return PGK_ERR_UNSUPPORTED;
    hipStream_t st = static_cast<hipStream_t>(stream);
    pgk::ReducePlan pl = pgk::plan_reduce_max(outer, red, inner, dtype, aligned16(X));
    // (too little room for the faster way's segments: whole blocks, if that takes no more than there is)
    const size_t room = workspace && !(reinterpret_cast<uintptr_t>(workspace) & 3u) ? workspace_bytes : 0;
    if (pl.partial_elems * 8 > room) {
        const pgk::ReducePlan blocks = pgk::plan_reduce_max_blocks(outer, red, inner, dtype, aligned16(X));
        if (blocks.blocks > 0 && blocks.partial_elems * 8 <= room) pl = blocks;
    }
    if (pl.blocks <= 0 || pl.blocks > 0x7fffffffLL) return PGK_ERR_UNSUPPORTED;
    float* pv = nullptr;
    int* pi = nullptr;
    if (pl.partial_elems) {
        // segment results (value, position) of the first pass
        if (!workspace || workspace_bytes < pl.partial_elems * 8 || (reinterpret_cast<uintptr_t>(workspace) & 3u))
            return PGK_ERR_WORKSPACE;
        pv = static_cast<float*>(workspace);
        pi = reinterpret_cast<int*>(pv + pl.partial_elems);
    }
    const hipError_t e = pgk::launch_reduce_max(pl, X, out, idx, pv, pi, outer, red, inner, dtype, st);
    return e == hipSuccess ? PGK_OK : PGK_ERR_HIP;
}

}  // extern "C"

namespace {

struct ConvPlan {
    bool valid;          // arguments make sense
    bool fast;           // matrix-core path
    int64_t Lout;
    // matrix-core path, where the B operand comes from:
    //   strips: the input itself; the tile columns whose reads would leave a row (listed in
    //           edge_tn) read zero-padded strips of edge_w columns instead;
    //   table:  stride * shifts copies of the input (see launch_conv_phase_copies), rows of Lq
    //           elements and cin_pad channels; tap k reads copy (k dil mod stride, h) at column
    //           offset (k dil div stride) - h, with h = 1 where that offset would be odd in bf16;
    //   else:   a zero-padded copy of the whole input with rows of Lp elements (Lp = 0: the
    //           input as it is -- no padding and aligned rows)
    //           (reg: tile bases off 4-byte boundaries -- bf16 with an odd dilation, padding or row
    //           length -- are copied through registers)
    bool strips, reg;
    int n_edges;
    int edge_tn[3];
    int edge_first_col[3];
    int64_t edge_w;
    int64_t Lp;
    bool table;
    int shifts;
    int64_t Lq, cin_pad;
    int kind;            // tile shape (TILE_*), chosen as for a plain GEMM of Cout x Lout
    pgk::TileShape tile;
    size_t w_bytes, x_bytes;   // workspace parts: regrouped weights; copies of the input or strips
    int in_place_rows;         // x read in place by tiles of so many output channels and 128 positions, whatever the rest says (0: not so);
                               // bf16 with `regrouped` bytes of workspace
    size_t regrouped;
};

size_t round_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// The kernels that read views of the input, or copies of it.
// no_copies: registers wherever there is a kernel for them (a workspace without room for copies of the input)
ConvPlan plan_conv_views(int64_t B, int64_t Cin, int64_t L, int64_t Cout, int64_t Kw, int64_t stride, int64_t pad,
                     int64_t dilation, int dtype, bool no_copies = false)
{
    ConvPlan pl{};
    if (B <= 0 || Cin <= 0 || L <= 0 || Cout <= 0 || Kw <= 0 || stride <= 0 || pad < 0 || dilation <= 0) return pl;
    if (dtype != PGK_DTYPE_F32 && dtype != PGK_DTYPE_BF16) return pl;
    if (B > kMaxDim || Cin > kMaxDim || L > kMaxDim || Cout > kMaxDim || Kw > kMaxDim || pad > kMaxDim ||
        dilation > kMaxDim || stride > kMaxDim) return pl;
    const int64_t span = L + 2 * pad - dilation * (Kw - 1) - 1;
    if (span < 0) return pl;
    pl.Lout = span / stride + 1;
    if (Cin * Kw > kMaxDim) return pl;
    pl.valid = true;
    const int64_t es = dtype == PGK_DTYPE_BF16 ? 2 : 4, epc = 16 / es;
    const pgk::TileShape t = pgk::mfma_tile_shape(dtype, false);
    // very short outputs stay with the bounds-checked kernel.  The output length may be anything
    // (the kernels store a row's last, partly filled chunk element by element), but the B copies
    // then reach up to Lr - 1 = the last column of that chunk, which the copies of the input must hold.
    if (pl.Lout < 16) return pl;
    const int64_t Lr = (int64_t)round_up((size_t)pl.Lout, (size_t)epc);
    // (up to 32 output channels: the flat tile, as for a GEMM with that many rows)
    pl.kind = Cout <= 32 ? pgk::TILE_FLAT : auto_tile_kind(Cout, pl.Lout, 0, dtype, B, false);
    pl.tile = pgk::mfma_tile_shape(dtype, pl.kind);
    const int64_t bn = pl.tile.bn, halo = (Kw - 1) * dilation;
    const bool shifts_even = dtype == PGK_DTYPE_F32 || dilation % 2 == 0 || Kw == 1;
    // (bf16: every tile base on a 4-byte boundary)
    const bool bases_even = shifts_even && (L * es) % 4 == 0 && (pad * es) % 4 == 0;
    // Otherwise tiles are copied through registers, or first into copies of the input (two shifted ones; a padded one where
    // the taps' offsets are even).  The registers cost 0.35 of the loop in the round model on the large tile, 0.5 on the small one, 0.7 on half
    // tiles, and 0.6 of a full round's with a single workgroup on a CU; the copies three passes over the input at 3.5 TB/s.
    // Fitted to 464 convolutions of up to 3000 products per output position and input channel (beyond, the copies): of the choices six are more
    // than 5 % slower than the copies, none than the registers.  Copies / registers: [8, 512, 4096] x [512, 512, 3] 66 / 58 us, [8, 128, 54071] x
    // [256, 128, 1] 193 / 103; [7, 384, 1656] x [265, 384, 10] 65 / 83, [2, 448, 576] x [234, 448, 5] 26 / 33.
    auto reg_pays = [&]() {
        const Rounds r = rounds_of(Cout, pl.Lout, dtype, B, pl.kind);
        const double loops = tile_cost(dtype, pl.kind).per_k * (double)Cin * (double)Kw / 1024.0 * (r.full + (r.rest == 1 ? 0.6 : r.rest > 1 ? 1.0 : 0.0));
        const double lost = pl.kind == pgk::TILE_LARGE ? 0.35 : pl.kind == pgk::TILE_SMALL ? 0.5 : 0.7;
        return lost * loops < 6.0 * (double)B * (double)Cin * (double)L / 3.5e6 + 1.5;
    };
    const bool reg = !bases_even && pl.kind != pgk::TILE_FLAT && Cout * Kw <= 3000 && (no_copies || reg_pays());
    // Reading the input in place needs the halo and the padding to be no wider than a tile.
    const bool strips = ((bases_even && (pl.Lout % epc == 0 || pl.kind != pgk::TILE_FLAT)) || reg) && halo <= bn && pad <= bn &&
                        (long double)B * Cin * 3 * ((bn + halo) / 256 + 2) < 2.0e9L;

    if (stride == 1 && Cin % t.bk == 0 && (shifts_even || strips)) {
        // the input as it is, or one zero-padded copy of it; taps a constant column step apart
        const int64_t K = Cin * Kw;
        const bool needs_copy = pad > 0 || L % epc != 0 || pl.Lout % epc != 0;
        const int64_t Lp = needs_copy ? (int64_t)round_up((size_t)std::max(L + 2 * pad, Lr + halo), (size_t)epc) : L;
        if ((int64_t)t.bm * K * es >= (1LL << 32) || (int64_t)t.bk * Lp * es + dilation * Kw * es >= (1LL << 32)) return pl;
        pl.fast = true;
        pl.w_bytes = round_up((size_t)(Cout * K * es), 256);
        pl.strips = strips;
        pl.reg = reg && strips;
        if (pl.strips) {
            const int64_t tiles_n = (pl.Lout + bn - 1) / bn;
            pl.edge_w = (int64_t)round_up((size_t)(bn + halo), (size_t)epc);
            pl.n_edges = 0;
            // (the last tile column reads whole 16-byte chunks, past the row's end where the output length is none)
            if (pad > 0 || pl.Lout % epc != 0) {
                const int64_t r0 = pl.Lout > pad ? (pl.Lout - pad) / bn : 0;     // first tile column reading past the end
                for (int64_t tn = 0; tn < tiles_n; ++tn)
                    if ((tn == 0 && pad > 0) || tn >= r0) {
                        pl.edge_tn[pl.n_edges] = (int)tn;
                        pl.edge_first_col[pl.n_edges] = (int)(tn * bn - pad);
                        ++pl.n_edges;
                    }
            }
            pl.x_bytes = round_up((size_t)pl.n_edges * (size_t)B * (size_t)Cin * (size_t)pl.edge_w * (size_t)es, 256);
            pl.Lp = 0;
        } else {
            pl.Lp = needs_copy ? Lp : 0;
            pl.x_bytes = needs_copy ? round_up((size_t)B * (size_t)Cin * (size_t)Lp * (size_t)es, 256) : 0;
        }
        return pl;
    }

    // Everything else with enough channels: stride > 1 (one copy per phase), a channel count
    // that is not a multiple of the K tile (copies and weights padded with zero channels), bf16
    // taps at odd column offsets (a second copy shifted by one element).  Each tap's place comes
    // from a table.  Padding the channels more than twofold would cost more than it gains.
    pl.cin_pad = (int64_t)round_up((size_t)Cin, (size_t)t.bk);
    if (Kw > pgk::kMaxTableTaps || pl.cin_pad > 2 * Cin) return pl;
    const int64_t K = pl.cin_pad * Kw;
    const int64_t q_max = halo / stride;
    pl.shifts = 1;
    if (dtype == PGK_DTYPE_BF16)
        for (int64_t k = 0; k < Kw; ++k)
            if ((k * dilation / stride) % 2 != 0) pl.shifts = 2;
    pl.Lq = (int64_t)round_up((size_t)(Lr + q_max + 1), (size_t)epc);
    if ((int64_t)t.bm * K * es >= (1LL << 32) || (int64_t)t.bk * pl.Lq * es >= (1LL << 32)) return pl;
    const long double copies_bytes = (long double)stride * pl.shifts * B * pl.cin_pad * pl.Lq * es;
    if (copies_bytes >= 4.0e12L || (long double)stride * pl.shifts * B * pl.cin_pad > 4.0e9L) return pl;
    pl.fast = true;
    pl.table = true;
    pl.w_bytes = round_up((size_t)(Cout * K * es), 256);
    pl.x_bytes = round_up((size_t)copies_bytes, 256);
    return pl;
}

// How long a grid of `wgs` workgroups takes whose K loops have `steps` steps of 32, in us: fixed + (steps + ends) times what a step takes
// a workgroup alone on its CU, or times `shared` for each of the CU's where these are more.
struct StepCost { double fixed, ends, alone, shared; int per_cu; };

double stepped_time(const StepCost& c, int64_t steps, double wgs)
{
    const double per = wgs / kNumCUs, on_busiest = per <= c.per_cu ? std::ceil(per) : per + 0.3;
    return c.fixed + ((double)steps + c.ends) * std::max(c.alone, c.shared * on_busiest);
}

// fp32: the input and the weights read in place (pgk_gemm_f32_terms.h, VIEW_INPUT), without a launch that copies or regroups,
// K = Cin * Kw without padding channels and tiles of 128, 64 or 32 output channels.  Bound like that kernel by issue slots, of which the loads take
// more than from a matrix, so that few workgroups with long sums are slower than the fp32 instruction's small tiles.  The constants
// were fitted to 400 drawn convolutions of strides 1 and 2 with each way forced, both off by a tenth in the root mean square: of the choices one is
// over 2 % slower than the views (what larger strides and more workgroups add: `apart` below), the mean is 1.21 times as fast, 0.97 of what the best way each time gives.  [10, 152, 53120] x
// [19, 152, 7] 450 us in the views, 305 here; [16, 57, 36868] x [67, 57, 5] 314 and 246; [2, 463, 2816] x [24, 463, 5], 46 workgroups and 73 steps,
// 51 and 82.  What has neither views nor enough to do for pgk_conv_few.hip was on the bounds-checked kernel: of 76 shapes none is
// slower here, the mean 1.27 times as fast.
int conv_rows_in_place(const ConvPlan& views, int64_t B, int64_t Cin, int64_t L, int64_t Cout, int64_t Kw, int64_t stride, int64_t pad,
                       int64_t dilation)
{
    // Sums of a few products: the three terms leave out up to 2^-24 of a product, which one product alone shows (worst error 1.4 to 1.7 x 2^-24
    // of it, a multiply-add's 1.0; root mean square 1.02 of that), and more of them hide behind the roundings that are spared: with
    // heavy-tailed values no later than at 12 (worst 0.7 to 0.9, root mean square 0.9 of a chain of multiply-adds; uniform 0.5 to 0.6).
    if (Cin * Kw < 12) return 0;
    // byte offsets inside a row with its padding, inside a batch entry, and inside a tile of the weights
    if (views.Lout < 16 || L + 2 * pad >= (1LL << 29) || Cin * L + pad >= (1LL << 30) - 4 || Cin * Kw * 128 >= (1LL << 30)) return 0;
    const int64_t tiles_n = (views.Lout + 127) / 128;
    auto wgs = [&](int64_t rows, int64_t tiles) { return (double)((Cout + rows - 1) / rows) * (double)tiles * (double)B; };
    if (wgs(32, tiles_n) > 2.0e9) return 0;
    const struct { int rows; StepCost cost; } kinds[] = {{128, {4.84, 2.28, 1.82, 1.37, 2}}, {64, {5.46, 1.31, 1.27, 0.88, 3}}, {32, {4.79, 1.18, 1.06, 0.66, 3}}};
    int best = 0;
    double best_time = 0.0;
    // A strided load takes a line for every few lanes, and starts its lanes on few of the cache's banks if the stride is even: so much more of a
    // step for each workgroup (with many on a CU, strides 2, 3, 4, 5 and 8: 0.26, 0.2, 0.9, 0.6 and 1.4, with one or two, which the
    // cache holds, less; [1, 256, 131200] x [19, 256, 10] stride 2 162 us in the views, 229 here).  Of 1200 drawn convolutions of strides 2 to
    // 11 without it 45 were over 5 % slower than before there was this way, 0.56 the worst.
    const double apart = (stride % 2 != 0 ? 0.11 : 0.2) * (double)(std::min<int64_t>(stride, 4) - 1);
    for (const auto& k : kinds) {
        StepCost cost = k.cost;
        cost.shared += apart;
        const double t = stepped_time(cost, (Cin * Kw + 31) / 32, wgs(k.rows, tiles_n));
        if (!best || t < best_time) { best = k.rows; best_time = t; }
    }
    if (!views.fast) return pgk::conv_few_channels_fits(B, Cin, Cout, Kw, stride, dilation, views.Lout) ? 0 : best;
    const bool copied = views.table || views.Lp > 0;
    const double copies = copied ? 0.17e-6 * 4.0 * (double)B * ((double)Cin * (double)L + (double)((Cin + 31) / 32 * 32) * (double)views.Lout * (double)stride) : 0.0;
    // (the views' large tile is this kernel too: equal within what the runs differ where nothing is copied or padded, [16, 64, 65536] x [128, 64, 3] 341
    // in the views, 345 here, with rows of 65538 360 and 340)
    const StepCost cost = views.kind == pgk::TILE_FLAT    ? StepCost{7.2, 2.0, 0.56, 0.56, 4}
                          : views.kind == pgk::TILE_SMALL ? StepCost{7.4, 1.7, 0.51, 0.51, 4}
                                                          : StepCost{7.0, 2.2, 1.89, 1.38, 2};
    const double in_views = copies + stepped_time(cost, Kw * ((Cin + 31) / 32), wgs(views.tile.bm, (views.Lout + views.tile.bn - 1) / views.tile.bn));
    return best_time < 0.97 * in_views ? best : 0;
}

// bf16: blocks of 32 channels of the input in LDS, position by position (pgk_conv_bf16.hip), without copies of the input, without a K loop through
// registers, and x read once for all taps.  A block takes what its loads and barriers take or, on a full CU, its taps and its
// rows for every workgroup; up to six of them a CU go in whole rounds.  The constants were fitted to 420 drawn convolutions, these and those of the
// views' kernels (both off by an eighth in the root mean square), and the line lies where few choices are wrong: of 2400 others, half of them with long
// sums, nine are over 5 % slower than before there was this way, 0.82 the worst (46 with the line at 0.92 of the views' time and without whole
// rounds, 0.63: [2, 665, 11631] x [392, 665, 10] stride 2 113 us, 180 here), the mean is 1.60 times as fast, 1.14 with long sums.  [13, 384, 11631] x [61, 384, 5]
// stride 2 117 us in the views, 58 here, [13, 64, 4673] x [128, 64, 7] stride 2 39 and 17; long sums over many channels are the views': [8, 512, 4096] x [512,
// 512, 3] 56 and 86.  From 16 channels on also what had no views, which is faster here throughout (89 of the 420): [13, 20, 26691] x [202, 20, 3] 287
// on the bounds-checked kernel and 63, [13, 17, 61760] x [64, 17, 1] 85 on the one for few channels and 27; the outputs' rounding covers what the
// matrix instruction's sums differ by (16 to 31 channels, 16 to 310 products, four kinds of data: error against 64 bits the same to six digits).
int conv_bf16_in_place(const ConvPlan& views, int64_t B, int64_t Cin, int64_t L, int64_t Cout, int64_t Kw, int64_t stride, int64_t pad, int64_t dilation)
{
    const int64_t blocks = (Cin + 31) / 32, tiles_n = (views.Lout + 127) / 128;
    if (views.Lout < 16 || Cin < 16 || L >= (1 << 27) || (long double)Cout * Kw * blocks * 64 >= 2.0e9L ||
        (long double)((tiles_n + 4) * 128) * stride + pad >= 2.0e9L || (long double)(Cout + 31) / 32 * tiles_n * B >= 2.0e9L) return 0;
    struct Cost { int rows, per_cu; double fixed, per_round, part, tap_alone, group_alone, tap, group; };
    const Cost kinds[] = {{128, 2, 6.90, 1.43, 0.19, 0.293, 0.37, 0.218, 0.25}, {64, 4, 6.47, 0.77, 0.24, 0.192, 0.31, 0.131, 0.173},
                          {32, 4, 5.90, 0.48, 0.31, 0.156, 0.31, 0.059, 0.142}};
    const int64_t groups = ((Kw - 1) * dilation + 127 * stride + 1 + 127) / 128;
    int best = 0;
    double best_time = 0.0;
    for (const Cost& k : kinds) {
        int parts = 1;
        const size_t lds = pgk::conv_bf16_lds(Kw, stride, dilation, L, k.rows, &parts);
        if (!lds) return 0;
        const double per = (double)((Cout + k.rows - 1) / k.rows) * (double)tiles_n * (double)B / kNumCUs;
        const double on_busiest = per <= std::max(6.0, std::min<double>(k.per_cu, (double)(160 * 1024 / lds))) ? std::ceil(per) : per + 0.3;
        const double t = k.fixed + k.per_round * on_busiest +
                         (double)blocks * std::max(k.tap_alone * (double)Kw + k.part * parts + k.group_alone * (double)groups,
                                                   on_busiest * (k.tap * (double)Kw + k.group * (double)groups));
        if (!best || t < best_time) { best = k.rows; best_time = t; }
    }
    if (!views.fast) return best;
    const double copies = views.table || views.Lp > 0 ? 0.21e-6 * 2.0 * (double)B * ((double)Cin * (double)L + (double)((Cin + 63) / 64 * 64) * (double)views.Lout * (double)(stride * std::max(views.shifts, 1))) : 0.0;
    const StepCost cost = views.kind == pgk::TILE_FLAT    ? StepCost{8.2, 0.0, 0.49, 0.43, 4}
                          : views.kind == pgk::TILE_SMALL ? StepCost{9.1, 4.5, 0.515, 0.423, 2}
                          : views.kind == pgk::TILE_LARGE ? StepCost{7.2, 7.7, 0.23, 1.235, 1}
                                                          : StepCost{6.5, 6.8, 0.79, 0.89, 1};
    const double wgs = (double)((Cout + views.tile.bm - 1) / views.tile.bm) * (double)((views.Lout + views.tile.bn - 1) / views.tile.bn) * (double)B;
    // (tiles of one to a CU: whole rounds)
    const double in_views = copies + stepped_time(cost, (int64_t)((double)(Kw * ((Cin + 63) / 64)) * (views.reg ? 1.38 : 1.0)),
                                                  cost.per_cu == 1 ? std::ceil(wgs / kNumCUs) * kNumCUs - (wgs > kNumCUs ? 0.3 * kNumCUs : 0.0) : wgs);
    return best_time < 0.85 * in_views ? best : 0;
}

ConvPlan plan_conv1d(int64_t B, int64_t Cin, int64_t L, int64_t Cout, int64_t Kw, int64_t stride, int64_t pad, int64_t dilation, int dtype,
                     bool no_copies = false)
{
    ConvPlan pl = plan_conv_views(B, Cin, L, Cout, Kw, stride, pad, dilation, dtype, no_copies);
    if (pl.valid)
        pl.in_place_rows = dtype == PGK_DTYPE_F32 ? conv_rows_in_place(pl, B, Cin, L, Cout, Kw, stride, pad, dilation)
                                                  : conv_bf16_in_place(pl, B, Cin, L, Cout, Kw, stride, pad, dilation);
    if (pl.in_place_rows && dtype == PGK_DTYPE_BF16) pl.regrouped = round_up((size_t)(Cout * Kw * ((Cin + 31) / 32 * 32) * 2), 256);
    return pl;
}

// What the call writes to: in place nothing but a bf16 kernel's regrouped weights, whatever the views would take.
size_t touched_workspace(const ConvPlan& pl)
{
    return !pl.valid ? 0 : pl.fast && !pl.in_place_rows ? pl.w_bytes + pl.x_bytes : pl.regrouped;
}

}  // namespace

extern "C" {

int64_t pgk_conv1d_out_len(int64_t L, int64_t Kw, int64_t stride, int64_t pad, int64_t dilation)
{
    if (L <= 0 || Kw <= 0 || stride <= 0 || pad < 0 || dilation <= 0) return 0;
    const int64_t span = L + 2 * pad - dilation * (Kw - 1) - 1;
    return span < 0 ? 0 : span / stride + 1;
}

size_t pgk_conv1d_workspace_bytes(int64_t B, int64_t Cin, int64_t L, int64_t Cout, int64_t Kw, int64_t stride,
                                  int64_t pad, int64_t dilation, int dtype)
{
    const ConvPlan pl = plan_conv1d(B, Cin, L, Cout, Kw, stride, pad, dilation, dtype);
    return !pl.valid ? 0 : pl.fast ? pl.w_bytes + pl.x_bytes : pl.regrouped;
}

size_t pgk_conv1d_workspace_least_bytes(int64_t B, int64_t Cin, int64_t L, int64_t Cout, int64_t Kw, int64_t stride,
                                        int64_t pad, int64_t dilation, int dtype)
{
    return touched_workspace(plan_conv1d(B, Cin, L, Cout, Kw, stride, pad, dilation, dtype));
}

int pgk_conv1d(const void* x, const void* w, const float* bias, void* y, int64_t B, int64_t Cin, int64_t L,
               int64_t Cout, int64_t Kw, int64_t stride, int64_t pad, int64_t dilation, int act, int dtype,
               void* workspace, size_t workspace_bytes, void* stream)
{
    if (!x || !w || !y) return PGK_ERR_INVALID_ARG;
    if (act < PGK_ACT_NONE || act > PGK_ACT_SILU) return PGK_ERR_INVALID_ARG;
    ConvPlan pl = plan_conv1d(B, Cin, L, Cout, Kw, stride, pad, dilation, dtype);
    if (!pl.valid) {
        // tell "out of range" from "makes no sense"
        if (B > 0 && Cin > 0 && L > 0 && Cout > 0 && Kw > 0 && stride > 0 && pad >= 0 && dilation > 0 &&
            (dtype == PGK_DTYPE_F32 || dtype == PGK_DTYPE_BF16) && pgk_conv1d_out_len(L, Kw, stride, pad, dilation) > 0)
            return PGK_ERR_UNSUPPORTED;
        return PGK_ERR_INVALID_ARG;
    }
    if (pl.fast && workspace && workspace_bytes < touched_workspace(pl)) {
        const ConvPlan in_place = plan_conv1d(B, Cin, L, Cout, Kw, stride, pad, dilation, dtype, true);
        if (in_place.fast && touched_workspace(in_place) <= workspace_bytes) pl = in_place;
    }
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int64_t es = dtype == PGK_DTYPE_BF16 ? 2 : 4;
    if ((long double)B * Cout * pl.Lout >= 4.6e18L || (long double)B * Cin * L >= 4.6e18L) return PGK_ERR_UNSUPPORTED;
    // The weights are always regrouped into the workspace, y and the bias may start on any element;
    // only an input that the kernels read in place has to start on a 16-byte boundary -- not where it is copied
    // through registers, which take any element, nor where the outputs are no whole chunks, whose tile bases lie off
    // that boundary anyway: the direct copies take 4-byte ones, the registers the rest.
    const bool reads_x_in_place = pl.strips || (!pl.table && pl.Lp == 0);
    const bool ragged_strips = pl.strips && pl.Lout % (16 / es) != 0;
    if (pl.fast && reads_x_in_place && !pl.reg && !aligned16(x)) {
        if (!ragged_strips) pl.fast = false;
        else if (reinterpret_cast<uintptr_t>(x) & 3u) pl.reg = true;
    }

    GemmArgs a{};
    a.bias = bias; a.C = y; a.ws = nullptr; a.rs_part = nullptr;
    a.M = (int)Cout; a.N = (int)pl.Lout; a.K = (int)(Cin * Kw); a.batch = (int)B;
    pgk::fill_plain_views(a);
    a.a_batch_stride = 0;                 // the weights are shared by the batch entries
    a.bias_per_row = 1;                   // one bias per output channel = per row
    a.act = act; a.splits = 1;

    if (const size_t least = touched_workspace(pl);
        pl.fast && least && (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255u) || workspace_bytes < least)) return PGK_ERR_WORKSPACE;
    // (bf16 that has no other use for a workspace: without one it stays on the bounds-checked kernel)
    if (pl.regrouped && workspace && !(reinterpret_cast<uintptr_t>(workspace) & 255u) && workspace_bytes >= pl.regrouped) {
        const int cin_pad = (int)((Cin + 31) / 32 * 32);
        if (pgk::launch_conv_repack_weights(w, workspace, (int)Cout, (int)Cin, cin_pad, (int)Kw, dtype, st) != hipSuccess) return PGK_ERR_HIP;
        return pgk::launch_conv_bf16(x, workspace, bias, y, B, (int)Cin, cin_pad, (int)L, (int)Cout, (int)Kw, (int)stride, (int)pad, (int)dilation,
                                     (int)pl.Lout, pl.in_place_rows, act, st) == hipSuccess ? PGK_OK : PGK_ERR_HIP;
    }
    if (pl.in_place_rows && dtype == PGK_DTYPE_F32) {
        const int64_t rows = pl.in_place_rows;
        a.A = w; a.B = x;
        a.b_batch_stride = Cin * L;
        a.ldb = (int)L;
        a.conv_kw = (int)Kw; a.conv_stride = (int)stride; a.conv_pad = (int)pad; a.conv_dil = (int)dilation; a.conv_len = (int)L;
        a.k_slice = (a.K + 31) / 32 * 32;
        a.tiles_m = (int)((Cout + rows - 1) / rows);
        a.tiles_n = (int)((pl.Lout + 127) / 128);
        a.group_m = group_m_for(a.tiles_m, a.tiles_n);
        return pgk::launch_conv_f32_terms(a, (int)rows, st) == hipSuccess ? PGK_OK : PGK_ERR_HIP;
    }
    if (pl.fast) {
        unsigned char* wr = static_cast<unsigned char*>(workspace);
        unsigned char* xp = wr + pl.w_bytes;
        const void* bsrc = x;
        int64_t ldb = L, cin_k = Cin;
        if (pl.table) {
            cin_k = pl.cin_pad;
            // the copies of the input and the regrouped, channel-padded weights in one launch
            if (pgk::launch_conv_phase_copies(x, xp, B, (int)Cin, (int)pl.cin_pad, (int)L, (int)pl.Lq, (int)pad, (int)stride,
                                              pl.shifts, w, wr, (int)Cout, (int)Kw, dtype, st) != hipSuccess) return PGK_ERR_HIP;
            bsrc = xp;
            ldb = pl.Lq;
            a.K = (int)(pl.cin_pad * Kw);
            a.b_use_tap_table = 1;
            const int64_t plane = B * pl.cin_pad * pl.Lq;          // elements of one copy
            for (int64_t k = 0; k < Kw; ++k) {
                const int64_t o = k * dilation, phase = o % stride, q = o / stride;
                const int64_t h = (pl.shifts == 2 && q % 2 != 0) ? 1 : 0;
                a.b_tap_off[k] = ((phase * pl.shifts + h) * plane + (q - h)) * es;
            }
        } else if (pl.strips) {
            // strips and regrouped weights in one launch
            if (pgk::launch_conv_prepare(x, xp, B * Cin, (int)L, (int)pl.edge_w, pl.n_edges, pl.edge_first_col, w, wr,
                                         (int)Cout, (int)Cin, (int)Kw, dtype, st) != hipSuccess) return PGK_ERR_HIP;
            if (pl.n_edges > 0) {
                for (int e = 0; e < pl.n_edges; ++e) {
                    a.edge_tn[e] = pl.edge_tn[e];
                    a.edge_B[e] = xp + (size_t)e * (size_t)(B * Cin) * (size_t)pl.edge_w * (size_t)es;
                }
                a.edge_ldb = (int)pl.edge_w;
                a.edge_batch_stride = Cin * pl.edge_w;
            }
            a.b_col_shift = -(int)pad;
        } else {
            if (pgk::launch_conv_repack_weights(w, wr, (int)Cout, (int)Cin, (int)Cin, (int)Kw, dtype, st) != hipSuccess)
                return PGK_ERR_HIP;
            if (pl.Lp) {
                if (pgk::launch_conv_pad_input(x, xp, B * Cin, (int)L, (int)pl.Lp, (int)pad, dtype, st) != hipSuccess)
                    return PGK_ERR_HIP;
                bsrc = xp;
                ldb = pl.Lp;
            }
        }
        const Path path = pl.reg ? Path{true, pl.kind, pl.tile}
                                 : choose_path(aligned16(wr) && (ragged_strips || aligned16(bsrc)), Cout, pl.Lout, cin_k * Kw, dtype, B, pl.kind, false, ldb);
        if (!path.mfma) return PGK_ERR_UNSUPPORTED;   // the plan has checked what the kernel needs
        a.A = wr; a.B = bsrc;
        a.a_batch_stride = 0;
        a.b_batch_stride = cin_k * ldb;
        a.ldb = (int)ldb;
        a.reg_b = pl.reg ? 1 : 0;
        a.b_tiles_per_tap = (int)(cin_k / path.tile.bk);
        a.b_tap_step = (int)dilation;
        a.k_slice = a.K;
        a.tiles_m = (int)((Cout + path.tile.bm - 1) / path.tile.bm);
        a.tiles_n = (int)((pl.Lout + path.tile.bn - 1) / path.tile.bn);
        if ((long double)a.tiles_m * a.tiles_n * B > 2.0e9L) return PGK_ERR_UNSUPPORTED;
        a.group_m = group_m_for(a.tiles_m, a.tiles_n);
        return pgk::launch_gemm_mfma(a, dtype, path.kind, 0, st) == hipSuccess ? PGK_OK : PGK_ERR_HIP;
    }
    // few input channels: a kernel of its own (conv_few_channels_fits says where the line lies and why);
    // what is left (long sums read in place because x is misaligned, short rows, little work) on the
    // bounds-checked kernel, also reading the input in place
    if (pgk::conv_few_channels_fits(B, Cin, Cout, Kw, stride, dilation, pl.Lout) &&
        (long double)((pl.Lout + 142) / 128) * ((Cout + 127) / 128) * B <= 2.0e9L)
        return pgk::launch_conv_few_channels(x, w, bias, y, B, (int)Cin, (int)L, (int)Cout, (int)Kw, (int)stride, (int)pad,
                                             (int)dilation, (int)pl.Lout, act, dtype, st) == hipSuccess ? PGK_OK : PGK_ERR_HIP;
    const pgk::TileShape t = pgk::guarded_tile_shape();
    a.A = w; a.B = x;
    a.b_batch_stride = Cin * L;
    a.conv_kw = (int)Kw; a.conv_stride = (int)stride; a.conv_pad = (int)pad; a.conv_dil = (int)dilation; a.conv_len = (int)L;
    a.k_slice = (int)(((a.K + t.bk - 1) / t.bk) * t.bk);
    a.tiles_m = (int)((Cout + t.bm - 1) / t.bm);
    a.tiles_n = (int)((pl.Lout + t.bn - 1) / t.bn);
    if ((long double)a.tiles_m * a.tiles_n * B > 2.0e9L) return PGK_ERR_UNSUPPORTED;
    a.group_m = group_m_for(a.tiles_m, a.tiles_n);
    return pgk::launch_gemm_guarded(a, dtype, 0, st) == hipSuccess ? PGK_OK : PGK_ERR_HIP;
}

int pgk_probe_mfma(int dtype, int random_operands, int iters, float* sink, double* flops_out, void* stream)
{
    if (!sink || iters < 1 || iters > (1 << 20)) return PGK_ERR_INVALID_ARG;
    if (dtype != PGK_DTYPE_F32 && dtype != PGK_DTYPE_BF16) return PGK_ERR_INVALID_ARG;
    const int workgroups = 2 * kNumCUs;
    if (flops_out) {
        const double per_instruction = dtype == PGK_DTYPE_BF16 ? 2.0 * 32 * 32 * 16 : 2.0 * 32 * 32 * 2;
        *flops_out = per_instruction * 32.0 * iters * 4.0 * workgroups;
    }
    const hipError_t e = pgk::launch_probe_mfma(dtype, random_operands != 0, iters, workgroups, sink,
                                                static_cast<hipStream_t>(stream));
    return e == hipSuccess ? PGK_OK : PGK_ERR_HIP;
}

int pgk_probe_mfma_fed(int copies, int iters, const void* src, size_t src_bytes, size_t resident_bytes,
                       int stream_every, uint64_t* clock_out, double* flops_out, void* stream)
{
    if (!clock_out || (reinterpret_cast<uintptr_t>(clock_out) & 7u)) return PGK_ERR_INVALID_ARG;
    if (iters < 2 || iters > (1 << 20) || (iters & 1) || stream_every < 0) return PGK_ERR_INVALID_ARG;
    const size_t piece = 65536;
    unsigned int resident = 1, streamed = 0;
    if (copies) {
        if (!src || !aligned16(src) || src_bytes < piece || src_bytes % piece != 0) return PGK_ERR_INVALID_ARG;
        if (resident_bytes < piece || resident_bytes % piece != 0 || resident_bytes > src_bytes) return PGK_ERR_INVALID_ARG;
        if (src_bytes / piece > 0x7fffffffu) return PGK_ERR_UNSUPPORTED;
        resident = (unsigned int)(resident_bytes / piece);
        streamed = (unsigned int)((src_bytes - resident_bytes) / piece);
    }
    if (flops_out) *flops_out = 2.0 * 32 * 32 * 16 * 32.0 * iters * 8.0 * kNumCUs;
    const hipError_t e = pgk::launch_probe_mfma_fed(copies != 0, iters, src, resident, streamed, stream_every,
                                                    reinterpret_cast<unsigned long long*>(clock_out),
                                                    static_cast<hipStream_t>(stream));
    return e == hipSuccess ? PGK_OK : PGK_ERR_HIP;
}

int pgk_probe_gemm_phases(const void* A, const void* B, const float* bias, void* C, float* rowsum_partials,
                          int64_t M, int64_t N, int64_t K, int act, int dtype, uint64_t* stamps, size_t stamps_bytes,
                          int32_t* workgroups_out, void* stream)
{
    int rc = validate_common(A, B, C, M, N, K, 1, act, dtype);
    if (rc != PGK_OK) return rc;
    if (!stamps || (reinterpret_cast<uintptr_t>(stamps) & 7u)) return PGK_ERR_INVALID_ARG;
    const pgk::TileShape t = pgk::mfma_tile_shape(dtype, pgk::TILE_LARGE);
    if (!aligned16(A) || !aligned16(B) || !mfma_shape_ok(M, N, K, dtype) || odd_rows(K, dtype, false, N).a ||
        odd_rows(K, dtype, false, N).b)
        return PGK_ERR_UNSUPPORTED;
    const int64_t tiles_m = (M + t.bm - 1) / t.bm, tiles_n = (N + t.bn - 1) / t.bn;
    if ((long double)tiles_m * tiles_n > 1.0e6L) return PGK_ERR_UNSUPPORTED;
    if (workgroups_out) *workgroups_out = (int32_t)(tiles_m * tiles_n);
    if (stamps_bytes < (size_t)(tiles_m * tiles_n) * pgk::kStampWords * sizeof(uint64_t)) return PGK_ERR_WORKSPACE;
    GemmArgs a{};
    a.A = A; a.B = B; a.bias = bias; a.C = C; a.rs_part = rowsum_partials;
    a.M = (int)M; a.N = (int)N; a.K = (int)K; a.batch = 1;
    pgk::fill_plain_views(a);
    mark_ragged_rows(a, dtype);
    a.act = act; a.splits = 1;
    a.k_slice = (int)(((K + t.bk - 1) / t.bk) * t.bk);
    a.tiles_m = (int)tiles_m; a.tiles_n = (int)tiles_n;
    a.group_m = group_m_for(a.tiles_m, a.tiles_n);
    a.stamps = reinterpret_cast<unsigned long long*>(stamps);
    return pgk::launch_gemm_mfma_timed(a, dtype, static_cast<hipStream_t>(stream)) == hipSuccess ? PGK_OK : PGK_ERR_HIP;
}

int pgk_probe_stream_read(const void* src, size_t bytes, float* sink, void* stream)
{
    if (!src || !sink || bytes == 0 || bytes % 16 || !aligned16(src)) return PGK_ERR_INVALID_ARG;
    const hipError_t e = pgk::launch_probe_stream_read(src, bytes, sink, static_cast<hipStream_t>(stream));
    return e == hipSuccess ? PGK_OK : PGK_ERR_HIP;
}

const char* pgk_status_string(int status)
{
    switch (status) {
    case PGK_OK: return "PGK_OK";
    case PGK_ERR_INVALID_ARG: return "PGK_ERR_INVALID_ARG: null pointer, non-positive size, or unknown act/dtype/splits";
    case PGK_ERR_UNSUPPORTED: return "PGK_ERR_UNSUPPORTED: size beyond the supported index range";
    case PGK_ERR_WORKSPACE: return "PGK_ERR_WORKSPACE: workspace missing, misaligned or too small";
    case PGK_ERR_HIP: return "PGK_ERR_HIP: the HIP runtime reported an error";
    default: return "PGK: unknown status";
    }
}

int pgk_version(void) { return 200; }

}  // extern "C"
