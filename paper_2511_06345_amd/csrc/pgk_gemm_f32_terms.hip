// fp32 GEMM kernels on the bf16 matrix cores: instances and launcher.  The kernel template is in
// pgk_gemm_f32_terms.h.
#include "pgk_gemm_f32_terms.h"

namespace pgk {

hipError_t launch_gemm_f32_terms(const GemmArgs& a, int out_mode, hipStream_t s)
{
    if (a.bias_per_row) return launch_terms<CfgTerms, VIEW_CONV>(a, out_mode, s);
    return a.b_trans ? launch_terms<CfgTermsT, VIEW_GEMM>(a, out_mode, s) : launch_terms<CfgTerms, VIEW_GEMM>(a, out_mode, s);
}

hipError_t launch_gemm_f32_terms_timed(const GemmArgs& a, hipStream_t s)
{
    return launch_terms<CfgTerms, VIEW_GEMM, true>(a, 0, s);
}

}  // namespace pgk
