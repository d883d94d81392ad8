// The wide verification GEMM on raw exponents (see gemm_prefill_kernel.inl).
#include "gemm_prefill_kernel.inl"

namespace cas {

int launch_gemm_prefill(cas_ctx* ctx, const VerifyArgs& a, int t) { return launch_wide<false>(ctx, a, t); }

bool gemm_wide_ok(const cas_ctx* ctx, int64_t rows, int64_t cols, int ncols) {
  return wide_shape_ok(ctx, rows, cols, (int)((cols + 31) / 32), ncols);
}

}  // namespace cas
