// Verification GEMM for 17 to 32 columns on the raw form: instantiates the forms of the kernel with two
// blocks of output columns
// (see gemm_verify_kernel.inl) in a translation unit of their own.
#include "gemm_verify_kernel.inl"

namespace cas {

int launch_gemm_verify_wide(cas_ctx* ctx, const VerifyArgs& a, int t) { return launch_verify<2, false>(ctx, a, t); }

}  // namespace cas
