// Matrix-core GEMM kernels for bf16 operands whose rows start on 2-byte boundaries only (an odd K;
// an odd N of a plain B; a convolution's taps at odd offsets): the instances whose copies go
// through registers, and their launcher.  The kernel template is in pgk_gemm_mfma_kernel.h.
#include "pgk_gemm_mfma_kernel.h"

namespace pgk {

namespace {
// The large tile has registers for one operand's pieces beside its accumulators, and not quite: of 256 five spill
// with B's pieces, eight in the convolution's form and sixteen with A's (scratch of 24, 36 and 68 bytes a lane).
// The small tile takes both operands that way, also where only one needs it; the half tiles have no such
// instances, as the small one is as fast or faster on what they are planned for (reg_tile_kind).
// With B through registers the A ring is two deep: the main loop then goes in trips of two K tiles instead of six (the rings'
// common period), which leaves at most four tiles to the loop's end, where loads are checked at run time, not eight.  The third stage gave A's
// direct copies more time, which does not show.  512 x 50257 x 768 70.9 -> 67 us, x 512 60.5 -> 55, 128 x 128 x 5443, 10 entries, 30.7 -> 22, 1000 x
// 2048 x 257 (B transposed) 16.0 -> 14.3, convolution [8, 512, 4096] x [512, 512, 3] 64 -> 61; 92 products and 14 convolutions: none over 1 % slower.
template <bool REG_A, bool REG_B>
using RegLarge = MfmaCfgReg<false, 256, 256, 64, 4, 2, REG_B ? 2 : 3, 2, REG_A, REG_B>;
template <bool BT>
using RegSmall = MfmaCfgReg<BT, 128, 128, 64, 2, 2, 2, 2, true, true>;
// (a convolution's weights are regrouped and always copied directly)
using ConvSmall = MfmaCfgReg<false, 128, 128, 64, 2, 2, 2, 2, false, true>;
using ConvTall = MfmaCfgReg<false, 256, 128, 64, 4, 2, 2, 2, false, true>;
using ConvWide = MfmaCfgReg<false, 128, 256, 64, 2, 4, 2, 2, false, true>;

}  // namespace

hipError_t launch_gemm_mfma_reg(const GemmArgs& a, int kind, int out_mode, hipStream_t s)
{
    const bool b_trans = a.b_trans != 0;
    if (a.bias_per_row) {
        if (b_trans || a.reg_a || out_mode != 0) return hipErrorInvalidValue;
        switch (kind) {
        case TILE_LARGE: return launch_cfg<RegLarge<false, true>, VIEW_CONV>(a, out_mode, s);
        case TILE_SMALL: return launch_cfg<ConvSmall, VIEW_CONV>(a, out_mode, s);
        case TILE_TALL: return launch_cfg<ConvTall, VIEW_CONV>(a, out_mode, s);
        case TILE_WIDE: return launch_cfg<ConvWide, VIEW_CONV>(a, out_mode, s);
        default: return hipErrorInvalidValue;
        }
    }
    if (kind == TILE_LARGE && !b_trans && !(a.reg_a && a.reg_b))
        return a.reg_a ? launch_cfg<RegLarge<true, false>, VIEW_GEMM>(a, out_mode, s)
                       : launch_cfg<RegLarge<false, true>, VIEW_GEMM>(a, out_mode, s);
    if (kind != TILE_SMALL) return hipErrorInvalidValue;
    return b_trans ? launch_cfg<RegSmall<true>, VIEW_GEMM>(a, out_mode, s) : launch_cfg<RegSmall<false>, VIEW_GEMM>(a, out_mode, s);
}

}  // namespace pgk
