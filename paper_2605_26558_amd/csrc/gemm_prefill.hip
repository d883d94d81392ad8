// The wide verification GEMM on raw exponents (see gemm_prefill_kernel.inl).
#include "gemm_prefill_kernel.inl"

namespace cas {

// X [ncols][cols] into the order in which the product reads it: per 16 columns, block of 128 values of k and pair of
// products a run of 64 lanes, lane (mi, mq) holding the operands of the two products (kBlockVals) for column mi.  Columns
// past ncols and k past cols are 0.  Read in place, the 16 rows of X that a fragment touches lay a power of two apart
// (8 KB at cols = 4096) and met in the same sets of the caches: the whole prompt of 508 tokens through 4 layers of the 8B
// shape took 7.7 ms instead of 5.3.
__global__ __launch_bounds__(256) void pack_x_kernel(const uint16_t* __restrict__ X, int ncols, int cols, int nblk,
                                                     uint4* __restrict__ out) {
  const int wave = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int mq = lane >> 4, n16 = wave / nblk, blk = wave - n16 * nblk, n = n16 * 16 + (lane & 15);
  if (n16 * 16 >= ncols) return;
  u32x4 w[4];  // positions 8 mq ..+7 of the block's four words
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int k = blk * 128 + 32 * j + 8 * mq;
    const uint16_t* src = X + (size_t)n * cols + k;
    w[j] = u32x4{0, 0, 0, 0};
    if (n >= ncols) continue;
    if (k + 8 <= cols) {
      __builtin_memcpy(&w[j], src, 16);
    } else {
#pragma unroll
      for (int i = 0; i < 8; ++i)
        if (k + i < cols) w[j][i >> 1] |= (uint32_t)src[i] << (16 * (i & 1));
    }
  }
  const uint32_t first = mq & 1 ? 0x07060302u : 0x05040100u, second = mq & 1 ? 0x05040100u : 0x07060302u;
#pragma unroll
  for (int i = 0; i < 4; ++i)
    out[((size_t)wave * 4 + i) * 64 + lane] =
        make_uint4(__builtin_amdgcn_perm(w[1][i], w[0][i], first), __builtin_amdgcn_perm(w[3][i], w[2][i], first),
                   __builtin_amdgcn_perm(w[1][i], w[0][i], second), __builtin_amdgcn_perm(w[3][i], w[2][i], second));
}

int launch_gemm_prefill(cas_ctx* ctx, const VerifyArgs& a, int t) { return launch_wide<false>(ctx, a, t); }

bool gemm_wide_ok(const cas_ctx* ctx, int64_t rows, int64_t cols) {
  return wide_shape_ok(ctx, rows, cols, (int)((cols + 31) / 32));
}

size_t gemm_wide_x_bytes(int64_t cols, int ncols) {
  return (size_t)((ncols + 15) / 16) * (size_t)((cols + 127) / 128) * 4096;
}

int launch_pack_x(cas_ctx* ctx, const uint16_t* X, int ncols, int cols, void* out) {
  const int nblk = (cols + 127) / 128, waves = (ncols + 15) / 16 * nblk;
  hipLaunchKernelGGL(pack_x_kernel, dim3((waves + 3) / 4), dim3(256), 0, ctx->stream, X, ncols, cols, nblk, (uint4*)out);
  CAS_HIP(ctx, hipGetLastError());
  return CAS_OK;
}

}  // namespace cas
