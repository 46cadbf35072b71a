// fp32 GEMM kernels on the bf16 matrix cores: instances and launcher.  The kernel template is in
// pgk_gemm_f32_terms.h.
#include "pgk_gemm_f32_terms.h"

namespace pgk {

hipError_t launch_gemm_f32_terms(const GemmArgs& a, int out_mode, hipStream_t s)
{
    if (a.bias_per_row) return launch_terms<CfgTerms, VIEW_CONV>(a, out_mode, s);
    return a.b_trans ? launch_terms<CfgTermsT, VIEW_GEMM>(a, out_mode, s) : launch_terms<CfgTerms, VIEW_GEMM>(a, out_mode, s);
}

hipError_t launch_conv_f32_terms(const GemmArgs& a, int rows, hipStream_t s)
{
    if (!a.bias_per_row || a.conv_kw <= 0 || a.splits != 1) return hipErrorInvalidValue;
    switch (rows) {
    case 128: return launch_terms<CfgTerms, VIEW_INPUT>(a, 0, s);
    case 64: return launch_terms<CfgTerms64, VIEW_INPUT>(a, 0, s);
    case 32: return launch_terms<CfgTerms32, VIEW_INPUT>(a, 0, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_gemm_f32_terms_timed(const GemmArgs& a, hipStream_t s)
{
    return launch_terms<CfgTerms, VIEW_GEMM, true>(a, 0, s);
}

}  // namespace pgk
