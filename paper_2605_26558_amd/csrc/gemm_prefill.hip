// The wide verification GEMM on raw exponents (see gemm_prefill_kernel.inl).
#include "gemm_prefill_kernel.inl"

namespace cas {

// X [ncols][cols] into the order in which the product reads it: per 16 columns and 32 values of k a run of
// 64 lanes, lane (mi, mq) holding k = 8 mq ..+7 of column mi.  Columns past ncols and k past
// cols are 0.  Read in place, the 16 rows of X that a fragment touches lay a power of two apart (8 KB at
// cols = 4096) and met in the same sets of the caches: the whole prompt
// of 508 tokens through 4 layers of the 8B shape took 7.7 ms instead of 5.3.
__global__ __launch_bounds__(256) void pack_x_kernel(const uint16_t* __restrict__ X, int ncols, int cols, int nk,
                                                     uint4* __restrict__ out) {
  const int wave = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int n16 = wave / nk, k = (wave - n16 * nk) * 32 + 8 * (lane >> 4), n = n16 * 16 + (lane & 15);
  if (n16 * 16 >= ncols) return;
  uint4 v = make_uint4(0, 0, 0, 0);
  if (n < ncols) {
    const uint16_t* src = X + (size_t)n * cols + k;
    if (k + 8 <= cols) {
      __builtin_memcpy(&v, src, 16);
    } else {
      uint16_t e[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) e[i] = k + i < cols ? src[i] : (uint16_t)0;
      __builtin_memcpy(&v, e, 16);
    }
  }
  out[(size_t)wave * 64 + lane] = v;
}

int launch_gemm_prefill(cas_ctx* ctx, const VerifyArgs& a, int t) { return launch_wide<false>(ctx, a, t); }

bool gemm_wide_ok(const cas_ctx* ctx, int64_t rows, int64_t cols) {
  return wide_shape_ok(ctx, rows, cols, (int)((cols + 31) / 32));
}

size_t gemm_wide_x_bytes(int64_t cols, int ncols) {
  return (size_t)((ncols + 15) / 16) * (size_t)((cols + 127) / 128) * 4096;
}

int launch_pack_x(cas_ctx* ctx, const uint16_t* X, int ncols, int cols, void* out) {
  const int nk = (cols + 127) / 128 * 4, waves = (ncols + 15) / 16 * nk;
  hipLaunchKernelGGL(pack_x_kernel, dim3((waves + 3) / 4), dim3(256), 0, ctx->stream, X, ncols, cols, nk, (uint4*)out);
  CAS_HIP(ctx, hipGetLastError());
  return CAS_OK;
}

}  // namespace cas
