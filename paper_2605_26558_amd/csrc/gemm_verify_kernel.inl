// Kernel template and launcher of the verification GEMM; gemm_verify.hip instantiates the forms
// for up to 16 columns, gemm_verify_wide.hip those for 17 to 32.
#pragma once
#include <algorithm>
#include "cas_device.hpp"
#include "cas_internal.hpp"

namespace cas {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

struct VerifyArgs {
  int rows, cols, bw, sw, lw, pw, ncols;
  const uint32_t* bitmap;
  const uint32_t* spec;
  const uint32_t* lo;
  const uint32_t* pruned;
  const uint16_t* X;  // [ncols][cols]
  float* Y;           // [ncols][yld] (epilogue 0)
  int yld;            // output rows per column in Y / out16 (>= rows: the launch may cover a block of rows)
  const uint8_t* sexp;  // shared-exponent form only: one exponent per bitmap word, ew bytes per row
  int ew;
  int epi;            // 0: Y = W X;  1: h = bf16(h + bf16(W X));  2: act[i] = swiglu(rows 2i, 2i+1)
  uint16_t* out16;    // h [ncols][yld] (epilogue 1) or act [ncols][yld/2] (epilogue 2)
};

constexpr int kFewGroups = 300;          // row groups below which a matrix gets more waves per row group
constexpr int kOneEach = 256;            // row groups up to which every CU of the whole card has one at most
constexpr int kNowhere = 0x7FFFF000;     // a byte offset past the records of every stream: reads as 0, fetches nothing
// A block of 16 rows x 128 columns in LDS: [1 + 32 positions][16 rows][4 words] values, position p of the four bitmap
// words of a row side by side (row 0 takes what lanes without a value left write).  Whatever positions the lanes of a
// wave are at, at most the two lanes that share a word of their position's row meet in a bank (such pairs are 5.0 of the
// 12.5 M cycles in which the LDS is active, 28672 x 4096 with 20 columns): with a row's values in
// column order the writes of the walks met in banks for 73 % of the cycles in which the LDS was active, and it was
// active for 79 % of the kernel's (28672 x 4096, 7 columns).  The four values that lie together are one lane's operand
// of a product; product kk takes position 8 mq + (kk ^ (mq & 1)) in lane group mq, so that the reads of two groups
// go to either half of the banks.
constexpr int kPosPitch = 64;
constexpr int kBlockVals = 33 * kPosPitch;

// A workgroup of Q waves owns 16 output rows and takes 128 Q columns per step.  Decode: wave w places the values of
// 16 / Q rows in a tile in LDS, a lane 32 columns of one row, so that a wave reads runs of 128 Q columns of each stream
// (460 bytes of spec, 150 of lo, 410 of pruned values at Q = 4, keep 600, t = 4).  Product: after a barrier wave w
// multiplies all 16 rows of its own block of 128 columns (part w of a row = blocks w, w + Q, ...) and goes on to the next
// step in the other tile.  Where every wave decoded the 16 x 128 block that it multiplied, the runs were a quarter as
// long and a line was fetched 1.4 times on average.  X goes from memory to the operand registers, eight consecutive
// columns per lane, word and load (which columns meet in a product is free as long as both operands agree): staged in
// LDS it cost a wave a round trip per staging with nothing else to do.  NB: blocks of 16 output columns (MFMA N = 16);
// every column is computed by the same operations whichever block and whatever company it has.  Products of 32 columns
// (16x16x32): twice the rate of 16x16x16, which the wide GEMM needs; here within 1 % for most sizes and 3 % slower at worst (16 columns, eight parts).  Mean relative error
// against 64 bits over 40 shapes of all sizes, the same parts in the same order: 1.455e-7, with products of 16 columns
// 1.459e-7; neighbours that cancel (4096 x 4096) 2.0e-8 and 2.2e-7, values spread over e^(4 sigma) 8.16e-9 and 8.17e-9,
// subnormal weights the same.  The parts of a row are added two by two and the pairs in order: one after the other, with the
// numbers of parts that went with it and products of 16 columns, 1.49e-7.
// Loads run half a step ahead: the pruned values of a step are fetched while its kept values are placed, the kept
// fields of the next step while the pruned values are placed; X of a step before its decode.  All are issued on every
// path: where a load may or may not have been issued, the wait for an older one waits for it as well.
// Measured, matrices read from HBM in turn, 1 / 7 / 20 columns, us: 28672 x 4096 59 / 63 / 79, 4096 x 14336 33 / 34 / 43, 6144 x
// 4096 20.6 / 21.1 / 25.3, 4096 x 4096 13.1 / 13.3 / 15.8, 128256 x 4096 244 / 261 / 329 (private tiles in column order and X
// through LDS: 71 / 85 / 116, 48 / 48 / 52, 22.5 / 25.4 / 34.0, 15.9 / 17.4 / 20.4, 308 / 332 / 422), 11003 x 5001 37 / 40 / 52
// (43 / 50 / 62).  28672 x 4096 with 7 columns is 4.0 TB/s; vector issue takes half of that
// time, and the loads of X (sixteen columns, 64 bytes of each) the 4 us between 1 and 7 columns.  Tried: lanes side by
// side reading a column together and handing the pieces on through ds_bpermute, the same (67.5 / 82); one tile and a
// second barrier instead of two tiles (five workgroups per CU instead of four), the same within 2 %.
template <int T, int Q, int NB, bool MX = false>
__global__ __launch_bounds__(64 * Q, 4) void gemm_verify_kernel(VerifyArgs a) {
  constexpr int WPR = 4 * Q;         // bitmap words per row and step = lanes per row
  constexpr int RPW = 64 / WPR;      // rows a wave decodes
  constexpr int BLOCK = kBlockVals + 64 / Q;  // values from block to block
  constexpr int TILE = Q * BLOCK;
  static_assert(RPW * Q == 16 && NB >= 1 && NB <= 2, "sixteen rows, at most two blocks of output columns");
  extern __shared__ uint16_t lds[];          // two tiles
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int row0 = blockIdx.x * 16;

  // ---- decode role: row r of the tile, word j of the step
  const int j = lane & (WPR - 1);
  const int r = wv * RPW + lane / WPR;
  const int rr = min(r, a.rows - 1 - row0);  // rows past the end repeat the last one
  auto rsrc = [&](const uint32_t* base, int words) {
    return __builtin_amdgcn_make_buffer_rsrc((void*)(base + (size_t)row0 * words), 0, 64 * words + 128, kRawBufferFlags);
  };
  const __amdgpu_buffer_rsrc_t rs_s = rsrc(a.spec, a.sw), rs_l = rsrc(a.lo, a.lw), rs_p = rsrc(a.pruned, a.pw);
  const int row_s = rr * a.sw * 4, row_l = rr * a.lw * 4, row_p = rr * a.pw * 4;
  const __amdgpu_buffer_rsrc_t rs_b = rsrc(a.bitmap, a.bw);
  const int row_b = rr * a.bw * 4;
  const __amdgpu_buffer_rsrc_t rs_e = __builtin_amdgcn_make_buffer_rsrc(  // of the exponent bytes
      MX ? (void*)(a.sexp + (size_t)row0 * a.ew) : nullptr, 0, MX ? 16 * a.ew : 0, kRawBufferFlags);
  uint16_t* const trow = lds + (j >> 2) * BLOCK + kPosPitch + r * 4 + (j & 3);

  // ---- product role: A[i = lane%16][four k of lane/16], B[k][n = lane%16]
  const int mi = lane & 15, mq = lane >> 4;
  const uint16_t* const a_even = lds + wv * BLOCK + (1 + 8 * mq + (mq & 1)) * kPosPitch + mi * 4;
  const uint16_t* const a_odd = a_even - 2 * (mq & 1) * kPosPitch;
  const uint32_t sel_even = mq & 1 ? 0x07060302u : 0x05040100u, sel_odd = mq & 1 ? 0x05040100u : 0x07060302u;
  // X is read through a descriptor that ends with its last word: words past it read as 0.  Columns of X (rows of the
  // array) that start in the middle of a word are read from the word's start on and shifted into place (align_x): a
  // 16-byte load that is not aligned to words takes its 64 lanes one by one.
  const int x_first = (int)(reinterpret_cast<uintptr_t>(a.X) >> 1) & 1;
  const __amdgpu_buffer_rsrc_t rs_x = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(a.X - x_first), 0, ((a.ncols * a.cols + x_first) * 2 + 3) & ~3, kRawBufferFlags);
  const bool x_odd = (a.cols & 1) || x_first;
  int x_off[NB];  // values in front of the column
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) x_off[nb] = x_first + (16 * nb + mi < a.ncols ? 16 * nb + mi : 0) * a.cols;

  f32x4 C[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) C[nb] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int nstep = (a.bw + WPR - 1) / WPR;
  uint32_t before = 0;  // kept values of the row before the step
  uint32_t m_next = 0, m = 0, p = 0;
  int e_next = 0, e = 0;
  auto load_mask = [&](int s) {
    const int w = s * WPR + j;  // past the end of the row: an offset past the records, which reads as 0
    m_next = __builtin_amdgcn_raw_buffer_load_b32(rs_b, w < a.bw ? row_b + w * 4 : kNowhere, 0, 0);
    if constexpr (MX) e_next = __builtin_amdgcn_raw_buffer_load_b8(rs_e, w < a.bw ? rr * a.ew + w : kNowhere, 0, 0);
  };
  KeptWindows<T, true, MX> kw;
  PrunedWindows pw;
  auto load_kept = [&](int s) {  // of the step whose mask came last
    m = m_next;
    e = e_next;
    const int cnt = __popc(m);
    int incl = cnt;
    incl += __builtin_amdgcn_update_dpp(0, incl, DPP_ROW_SHR1, 0xf, 0xf, false);
    incl += __builtin_amdgcn_update_dpp(0, incl, DPP_ROW_SHR2, 0xf, 0xf, false);
    incl += __builtin_amdgcn_update_dpp(0, incl, DPP_ROW_SHR4, 0xf, 0xf, false);
    incl += __builtin_amdgcn_update_dpp(0, incl, DPP_ROW_SHR8, 0xf, 0xf, false);
    if constexpr (Q >= 8) incl += __builtin_amdgcn_update_dpp(0, incl, DPP_ROW_BCAST15, 0xa, 0xf, false);
    if constexpr (Q == 16) incl += __builtin_amdgcn_update_dpp(0, incl, DPP_ROW_BCAST31, 0xc, 0xf, false);
    const bool in = s * WPR + j < a.bw;  // words past the end of the row have no fields
    p = before + (uint32_t)(incl - cnt);
    before += (uint32_t)__builtin_amdgcn_ds_bpermute((lane | (WPR - 1)) * 4, incl);
    kw.load(in ? p : 0u, rs_s, in ? row_s : kNowhere, rs_l, in ? row_l : kNowhere);
  };

  // X of the step: positions 8 mq ..+7 of word g of the wave's block
  u32x4 xf[NB][4];
  uint32_t xe[NB];  // the word behind the block
  auto load_x = [&](int s) {
    const int blk = (s * Q + wv) * 128;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const int off = ((x_off[nb] + blk) & ~1) * 2;
#pragma unroll
      for (int g = 0; g < 4; ++g) xf[nb][g] = __builtin_amdgcn_raw_buffer_load_b128(rs_x, off + 16 * mq + 64 * g, 0, 0);
      if (x_odd) xe[nb] = __builtin_amdgcn_raw_buffer_load_b32(rs_x, off + 256, 0, 0);
    }
  };
  // the word behind a lane's piece is the first of the lane 16 on, or of the next piece
  auto align_x = [&]() {
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int x_sh = (x_off[nb] & 1) * 16;
        u32x4& f = xf[nb][g];
        const uint32_t mine = mq ? f.x : g < 3 ? xf[nb][g < 3 ? g + 1 : 3].x : xe[nb];
        const uint32_t next = (uint32_t)__builtin_amdgcn_ds_bpermute(((lane + 16) & 63) * 4, (int)mine);
        f.x = __builtin_amdgcn_alignbit(f.y, f.x, x_sh);
        f.y = __builtin_amdgcn_alignbit(f.z, f.y, x_sh);
        f.z = __builtin_amdgcn_alignbit(f.w, f.z, x_sh);
        f.w = __builtin_amdgcn_alignbit(next, f.w, x_sh);
      }
  };
  // zeros past the last column
  auto trim_x = [&](int s) {
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int left = a.cols - ((s * Q + wv) * 128 + 32 * g + 8 * mq);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          if (left < 2 * i + 2) xf[nb][g][i] &= 0xFFFFu;
          if (left < 2 * i + 1) xf[nb][g][i] = 0;
        }
      }
  };

  load_mask(0);
  load_kept(0);
  load_mask(1);
  for (int s = 0; s < nstep; ++s) {
    uint16_t* const dst = trow + (s & 1) * TILE;
    const int nvalid = a.cols - (s * WPR + j) * 32;
    const uint32_t valid = nvalid >= 32 ? 0xFFFFFFFFu : (nvalid <= 0 ? 0u : ((1u << nvalid) - 1u));
    if (nvalid < 32) {  // columns past the end are not placed below
#pragma unroll
      for (int q = 0; q < 32; ++q) dst[q * kPosPitch] = 0;
    }
    load_x(s);
    pw.load(nvalid > 0 ? (uint32_t)(s * WPR + j) * 32u - p : 0u, rs_p, nvalid > 0 ? row_p : kNowhere);
    const uint32_t pm = ~m & valid;
    kw.decode(m, [&](int pos, uint16_t v) { dst[pos * kPosPitch] = v; }, MX ? e : 0);
    load_kept(s + 1);
    load_mask(s + 2);
    pw.decode(pm, [&](int pos, uint16_t v) { dst[pos * kPosPitch] = v; });
    __syncthreads();
    if (x_odd) align_x();
    if ((s * Q + wv) * 128 + 128 > a.cols) trim_x(s);
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const u32x2 a0 = *reinterpret_cast<const u32x2*>(a_even + (s & 1) * TILE + 2 * w * kPosPitch);
      const u32x2 a1 = *reinterpret_cast<const u32x2*>(a_odd + (s & 1) * TILE + (2 * w + 1) * kPosPitch);
      const bf16x8 av = __builtin_bit_cast(bf16x8, u32x4{a0.x, a0.y, a1.x, a1.y});
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        const u32x4* f = xf[nb];
        const u32x4 bv = {__builtin_amdgcn_perm(f[1][w], f[0][w], sel_even), __builtin_amdgcn_perm(f[3][w], f[2][w], sel_even),
                          __builtin_amdgcn_perm(f[1][w], f[0][w], sel_odd), __builtin_amdgcn_perm(f[3][w], f[2][w], sel_odd)};
        C[nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, __builtin_bit_cast(bf16x8, bv), C[nb], 0, 0, 0);
      }
    }
  }

  // ---- add the Q partial tiles of each row group, pairs of parts in order; C[i][n]: i = 4*(lane/16) + e, n = lane%16
  __syncthreads();
  float* red = reinterpret_cast<float*>(lds);  // [NB][Q][64][4], reuses the tiles
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) *reinterpret_cast<f32x4*>(red + ((nb * Q + wv) * 64 + lane) * 4) = C[nb];
  __syncthreads();
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    const int col = 16 * nb + mi;
    if (wv != 0 || col >= a.ncols) continue;
    auto part = [&](int w) { return *reinterpret_cast<f32x4*>(red + ((nb * Q + w) * 64 + lane) * 4); };
    f32x4 s = part(0) + part(1);
#pragma unroll
    for (int w = 2; w < Q; w += 2) s += part(w) + part(w + 1);
    if (a.epi == 0) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        int orow = row0 + 4 * mq + e;
        if (orow < a.rows) a.Y[(size_t)col * a.yld + orow] = s[e];
      }
    } else if (a.epi == 1) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        int orow = row0 + 4 * mq + e;
        if (orow < a.rows) {
          uint16_t* hp = a.out16 + (size_t)col * a.yld + orow;
          *hp = f32_to_bf16(bf16_to_f32(*hp) + round_bf16(s[e]));
        }
      }
    } else {  // rows come in (gate, up) pairs; a lane holds rows 4*mq .. 4*mq+3 = two pairs
#pragma unroll
      for (int e = 0; e < 4; e += 2) {
        int orow = row0 + 4 * mq + e;
        if (orow + 1 < a.rows) {
          const float g = round_bf16(s[e]), u = round_bf16(s[e + 1]);
          a.out16[(size_t)col * (a.yld >> 1) + (orow >> 1)] = f32_to_bf16(g / (1.0f + expf(-g)) * u);
        }
      }
    }
  }
}

template <int Q, int NB, bool MX = false>
static int launch_q(cas_ctx* ctx, const VerifyArgs& a, int t) {
  constexpr size_t lds = sizeof(uint16_t) * 2 * Q * (kBlockVals + 64 / Q);
  static_assert(lds >= sizeof(float) * NB * Q * 64 * 4, "the partial sums reuse the tiles");
  if (lds > (size_t)ctx->lds_max) return CAS_ENOTSUP;
  const int grid = (a.rows + 15) / 16;
#define CAS_LAUNCH(TV)                                                                                        \
  case TV: {                                                                                                  \
    static LdsLimit lim;                                                                                      \
    const int rc = allow_lds(ctx, (const void*)gemm_verify_kernel<TV, Q, NB, MX>, lds, lim);                  \
    if (rc != CAS_OK) return rc;                                                                              \
    hipLaunchKernelGGL((gemm_verify_kernel<TV, Q, NB, MX>), dim3(grid), dim3(64 * Q), lds, ctx->stream, a);    \
  } break;
  switch (t) {
    CAS_LAUNCH(0) CAS_LAUNCH(1) CAS_LAUNCH(2) CAS_LAUNCH(3) CAS_LAUNCH(4) CAS_LAUNCH(5) CAS_LAUNCH(6) CAS_LAUNCH(7)
    default: return CAS_EINVAL;
  }
#undef CAS_LAUNCH
  CAS_HIP(ctx, hipGetLastError());
  return CAS_OK;
}

// Waves per row group = parts that a row's columns are cut into.  The choice depends on the shape of the WHOLE matrix
// (not on the number of columns, on the form of the weights, on the block of rows a launch covers or on how many CUs a
// partition of the card has): it fixes the order in which a row's partial sums are added, and a column must get the same
// bits in every call.  Four where the row groups fill the chip (a step is then shortest and the barrier waits for the fewest
// waves) and for rows that one step of theirs covers.  Else more, so that each CU has waves to switch between: sixteen where
// a CU has one group and rounding up to whole steps costs a ninth at most, that is no half of one, or one half of five or more.
// Matrices read in turn, 4 / 8 / 16 waves, us, for 5 and for 20 columns: 4096 rows of 512 columns 4.4 / 5.4 / 7.1, 4.8 / 6.6 /
// 9.4; 1024 6.6 / 5.8 / 7.7, 7.1 / 6.9 / 10.2; 2048 10.2 / 8.7 / 8.3, 11.2 / 10.4 / 10.4; 3072 13.6 / 11.6 / 12.8, 15.6 / 13.8 /
// 16.3; 4096 17.1 / 14.2 / 13.0, 18.8 / 16.3 / 16.0; 7168 27.3 / 21.6 / 21.8, 31.3 / 26.2 / 27.5; 14336 49.7 / 38.9 / 35.2, 58.7 /
// 47.5 / 43.8; 1024 rows of 4096 15.5 / 12.0 / 11.3, 19.0 / 15.7 / 15.0, of 5120 18.8 / 14.3 / 15.3, 23.0 / 18.8 / 20.5; 4700 rows
// (294 groups) of 4096 20.9 / 20.2 / 22.4, 26.1 / 25.7 / 28.8; 6144 rows of 4096 21.4 / 21.1 / 22.9, 26.0 / 25.9 / 29.0.  Two
// sides on which the line does not lie best: 1025 to 1536 columns with 17 output columns or more (4096 x 1536, 20: 9.3 / 10.5
// / 10.4), and shared exponents from kFewGroups on (8192 x 4096, 5: 26.6 / 23.9 / 26.0; 8192 x 8192 48.5 / 43.5 / 46.3).  Sixteen
// waves (128 registers each) are all that a CU holds of this kernel, two workgroups of eight the same: where several streams
// verify at once, eight leave more to switch between.  us a product, one / two / three streams, 16 parts: 4096 x 4096 13.7 / 11.2 /
// 11.5, with 8 14.1 / 9.5 / 9.5; 1024 x 4096 11.3 / 6.0 / 4.4, with 8 12.4 / 7.2 / 5.2.  A pass
// that verifies several sequences is one launch, so the line is that of one stream.
static inline int verify_parts(int64_t rows, int64_t cols) {
  const int64_t groups = (rows + 15) / 16, steps8 = (cols + 1023) / 1024, steps16 = (cols + 2047) / 2048;
  if (groups >= kFewGroups || cols <= 512) return 4;
  return groups <= kOneEach && 9 * steps16 <= 5 * steps8 ? 16 : 8;
}

template <int NB, bool MX>
static int launch_verify(cas_ctx* ctx, const VerifyArgs& a, int t) {
  switch (verify_parts(a.yld, a.cols)) {
    case 4: return launch_q<4, NB, MX>(ctx, a, t);
    case 8: return launch_q<8, NB, MX>(ctx, a, t);
    default: return launch_q<16, NB, MX>(ctx, a, t);
  }
}

// gemm_verify_wide.hip: launch_verify<2, false> (its own translation unit: the build compiles the files side by side)
int launch_gemm_verify_wide(cas_ctx* ctx, const VerifyArgs& a, int t);
// gemm_prefill.hip, gemm_prefill_mx.hip: the form for the columns of a prompt
int launch_gemm_prefill(cas_ctx* ctx, const VerifyArgs& a, int t);
int launch_gemm_prefill_mx(cas_ctx* ctx, const VerifyArgs& a, int t);

}  // namespace cas
