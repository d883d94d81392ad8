// The wide verification GEMM on the shared-exponent form (see gemm_prefill_kernel.inl).
#include "gemm_prefill_kernel.inl"

namespace cas {

int launch_gemm_prefill_mx(cas_ctx* ctx, const VerifyArgs& a, int t) { return launch_wide<true>(ctx, a, t); }

}  // namespace cas
