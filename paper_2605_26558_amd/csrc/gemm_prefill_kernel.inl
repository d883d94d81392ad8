// Kernel template and launcher of the wide verification GEMM: the product of the exact matrix with the
// columns of a long prompt.  The verification GEMM decodes the matrix once per 32 columns at most; here a
// workgroup decodes 16 RT rows once for 256 columns.  Every output has the bits of the verification GEMM:
// the parts a row's columns are cut into, the order of the 32-column products within a part and the order
// in which the parts are added are the same.
#pragma once
#include <algorithm>
#include "gemm_verify_kernel.inl"

namespace cas {

constexpr int kWideThreads = 512;
constexpr int kWideCols = 256;  // columns of X per workgroup
constexpr int kXcds = 8;
constexpr int kAhead = 5;        // fragments of rows in registers ahead of their products

// bytes of the counts in front of every run of blocks
template <int RT>
__host__ __device__ constexpr size_t wide_pre_bytes(int bw) {
  constexpr int words = 4 * (8 / RT);  // of a run
  return (sizeof(uint16_t) * 16 * RT * (size_t)((bw + words - 1) / words) + 15) / 16 * 16;
}

// One workgroup per CU (8 waves of up to 256 registers).  A step takes a run of KB blocks of 128 columns, one block of
// each of KB parts: thread (row r, word j) places its 32 values in a tile in LDS, each wave multiplies all rows of the tile
// with its own NB blocks of 16 columns of X, n and n + 128, which it reads from memory (no other wave of the workgroup needs
// them), a running sum per part.  NB = 1 where the launch has no more than 128 columns (see launch_wide_rt).  Two tiles: while one is multiplied the next one is filled, with one barrier per step; the
// waves w and w + 4, which share a SIMD, take the two halves of a step in opposite order, so that the decode of
// the one runs under the matrix operations of the other.  Steps come by KB parts at a time (part p of Q has the blocks
// p, p + Q, ...); the sums of parts that are complete lie in LDS, the counts of kept values in front of every run of
// every row are made at the start (pre).
// Bound by memory, by what leaves the L2s and by the order in which loads come back.  28672 x 4096 with 508 columns: 1.47
// GB from behind the L2s and 368 us, where blocks came part by part (runs of 115 bytes of spec) and the workgroups of a row
// group went to different XCDs; 0.80 GB with these on one XCD, 0.59 with runs of KB blocks as well.  A prompt of 509 tokens
// through four layers, ms: 3.88 before; workgroups of a row group on one XCD 3.57 for 3.77; runs of KB blocks 3.47; loads
// issued on every path and no copy of a value in flight, so that no wait is for more than its own load, 3.41; five fragments
// ahead instead of three 3.40; 368 us are 317 then.  X of two blocks ahead instead of one is the same, products of 16 columns 3.57.
template <int T, int RT, int NB, bool MX>
__global__ __launch_bounds__(kWideThreads) void gemm_prefill_kernel(VerifyArgs a, int Q) {
  constexpr int ROWS = 16 * RT, KB = 128 / ROWS;
  static_assert(NB == 1 || NB == 2, "a wave has one block of columns, or two");
  static_assert(KB == 2 || KB == 4, "the fragments of X alternate between two sets");
  constexpr int BLOCK = RT * kBlockVals + 64 / KB;  // values from a block of 128 columns to the next: in other banks
  constexpr int TILE = KB * BLOCK;
  extern __shared__ uint16_t lds[];
  uint16_t* pre = lds + 2 * TILE;  // [ROWS][nrun] kept values of the row before each run of KB blocks
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ncb = (a.ncols + kWideCols - 1) / kWideCols;
  // workgroups go to the XCDs in turn: those of a row group, which read the same matrix, go to one
  const int on_xcd = (int)blockIdx.x / kXcds;
  const int cb0 = on_xcd % ncb * kWideCols, row0 = (on_xcd / ncb * kXcds + (int)blockIdx.x % kXcds) * ROWS;
  if (row0 >= a.rows) return;
  const int nblk = (a.bw + 3) >> 2, nrun = (nblk + KB - 1) / KB;
  const int per_part = (nblk + Q - 1) / Q;  // blocks of a part: part p has the blocks p, p + Q, ...
  const int nsteps = (min(Q, nblk) + KB - 1) / KB * per_part;  // a step takes a block of each of KB parts; parts without any come last

  // ---- kept values in front of every run
  {
    constexpr int RW = ROWS / 8;  // rows per wave
    uint32_t run[RW];
#pragma unroll
    for (int i = 0; i < RW; ++i) run[i] = 0;
    for (int w0 = 0; w0 < a.bw; w0 += 64) {
      uint32_t m[RW];
#pragma unroll
      for (int i = 0; i < RW; ++i) {
        const int row = min(row0 + wv * RW + i, a.rows - 1);
        m[i] = w0 + lane < a.bw ? a.bitmap[(size_t)row * a.bw + w0 + lane] : 0u;
      }
#pragma unroll
      for (int i = 0; i < RW; ++i) {
        const int cnt = __popc(m[i]), incl = wave_incl_scan(cnt);
        const int w = w0 + lane;
        if (w % (4 * KB) == 0 && w < a.bw) pre[(wv * RW + i) * nrun + w / (4 * KB)] = (uint16_t)(run[i] + (uint32_t)(incl - cnt));
        run[i] += (uint32_t)__builtin_amdgcn_readlane(incl, 63);
      }
    }
    __syncthreads();
  }

  // first bitmap word of a step; steps whose run lies past the end of the rows have no words
  auto step_word = [&](int st) -> int {
    const int g = st / per_part;
    return 4 * ((st - g * per_part) * Q + g * KB);
  };

  // ---- decode role: row r of the tile, word j of the step's run
  const int r = tid / (4 * KB), j = lane & (4 * KB - 1);
  const int row = min(row0 + r, a.rows - 1);
  auto rsrc = [&](const uint32_t* base, int words) {
    return __builtin_amdgcn_make_buffer_rsrc((void*)(base + (size_t)row0 * words), 0, ROWS * 4 * words + 128, kRawBufferFlags);
  };
  const __amdgpu_buffer_rsrc_t rs_s = rsrc(a.spec, a.sw), rs_l = rsrc(a.lo, a.lw), rs_p = rsrc(a.pruned, a.pw);
  const __amdgpu_buffer_rsrc_t rs_b = rsrc(a.bitmap, a.bw);
  const int rr = row - row0, row_s = rr * a.sw * 4, row_l = rr * a.lw * 4, row_p = rr * a.pw * 4, row_b = rr * a.bw * 4;
  const __amdgpu_buffer_rsrc_t rs_e = __builtin_amdgcn_make_buffer_rsrc(  // of the exponent bytes
      MX ? (void*)(a.sexp + (size_t)row0 * a.ew) : nullptr, 0, MX ? ROWS * a.ew : 0, kRawBufferFlags);
  uint16_t* const trow = lds + (j >> 2) * BLOCK + (r >> 4) * kBlockVals + kPosPitch + (r & 15) * 4 + (j & 3);
  WordWindows<T, true, MX> ww;
  uint32_t m_next = 0, m_cur = 0;
  int e_next = 0, e_cur = 0, nvalid = 0;
  // Loads are issued on every path, past the last step for that step again: where a load may or may not
  // have been issued, the compiler's wait for an older one waits for it as well.
  auto load_mask = [&](int st) {
    const int w = step_word(min(st, nsteps - 1)) + j;
    m_next = __builtin_amdgcn_raw_buffer_load_b32(rs_b, w < a.bw ? row_b + w * 4 : kNowhere, 0, 0);
    if constexpr (MX) e_next = __builtin_amdgcn_raw_buffer_load_b8(rs_e, w < a.bw ? rr * a.ew + w : kNowhere, 0, 0);
  };
  auto issue = [&](int st) {  // windows of the step whose mask came last
    const int w0 = step_word(min(st, nsteps - 1));
    m_cur = taken(m_next);
    if constexpr (MX) e_cur = (int)taken((uint32_t)e_next);
    const int cnt = __popc(m_cur);
    int incl = cnt;  // over the 4 KB lanes of a row
    if constexpr (KB == 4) {
      incl += __builtin_amdgcn_update_dpp(0, incl, DPP_ROW_SHR1, 0xf, 0xf, false);
      incl += __builtin_amdgcn_update_dpp(0, incl, DPP_ROW_SHR2, 0xf, 0xf, false);
      incl += __builtin_amdgcn_update_dpp(0, incl, DPP_ROW_SHR4, 0xf, 0xf, false);
      incl += __builtin_amdgcn_update_dpp(0, incl, DPP_ROW_SHR8, 0xf, 0xf, false);
    } else {
      const int b0 = quad_dpp<0x00>(cnt), b1 = quad_dpp<0x55>(cnt), b2 = quad_dpp<0xAA>(cnt);
      incl += ((j & 3) > 0 ? b0 : 0) + ((j & 3) > 1 ? b1 : 0) + ((j & 3) > 2 ? b2 : 0);
      const int quad = quad_dpp<0xFF>(incl);
      incl += __builtin_amdgcn_update_dpp(0, quad, DPP_ROW_SHR4, 0xf, 0xa, false);
    }
    nvalid = a.cols - (w0 + j) * 32;
    // words past the end of the row have no fields: keep their (unused) windows in range
    const uint32_t p = nvalid > 0 ? pre[r * nrun + w0 / (4 * KB)] + (uint32_t)(incl - cnt) : 0u;
    ww.k.load(p, rs_s, row_s, rs_l, row_l);
    ww.pr.load(nvalid > 0 ? (uint32_t)(w0 + j) * 32u - p : 0u, rs_p, row_p);
  };
  auto decode = [&](int st) {
    if (st < nsteps) {
      uint16_t* dst = trow + (st & 1) * TILE;
      const uint32_t valid = nvalid >= 32 ? 0xFFFFFFFFu : (nvalid <= 0 ? 0u : ((1u << nvalid) - 1u));
      if (nvalid < 32) {  // columns past the end are not placed below
#pragma unroll
        for (int q = 0; q < 32; ++q) dst[q * kPosPitch] = 0;
      }
      ww.decode(m_cur, ~m_cur & valid, [&](int pos, uint16_t v) { dst[pos * kPosPitch] = v; }, MX ? e_cur : 0);
    }
    issue(st + 1);
    load_mask(st + 2);
  };

  // ---- product role: columns cb0 + 16 wv + mi and 128 further; A[i = lane%16][k = 4*(lane/16)..+3]
  const int mi = lane & 15, mq = lane >> 4;
  const bool act0 = cb0 + 16 * wv < a.ncols, act1 = cb0 + 128 + 16 * wv < a.ncols;
  // X comes packed (pack_x_kernel): the fragments of 16 columns and 32 values of k are one run of 1 KB
  const size_t xrow = (size_t)nblk * 4 * 512;  // values of a block of 16 columns
  const uint16_t* const xp0 = a.X + (size_t)((cb0 >> 4) + (act0 ? wv : 0)) * xrow;
  auto rsrc_x = [&](const uint16_t* x) {
    return __builtin_amdgcn_make_buffer_rsrc((void*)x, 0, (int)(xrow * 2), kRawBufferFlags);
  };
  const __amdgpu_buffer_rsrc_t rs_x0 = rsrc_x(xp0), rs_x1 = rsrc_x(act1 ? xp0 + 8 * xrow : xp0);
  f32x4 C[KB][RT][NB];  // running sums of KB parts
#pragma unroll
  for (int jb = 0; jb < KB; ++jb)
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) C[jb][i][nb] = f32x4{0.f, 0.f, 0.f, 0.f};
  // sum of the parts before them, in LDS: touched once in per_part steps
  f32x4* const S = reinterpret_cast<f32x4*>(reinterpret_cast<char*>(pre) + wide_pre_bytes<RT>(a.bw)) + wv * (RT * NB * 64) + lane;
  uint4 x[4][NB];  // of one block; zeros for one past the end of the rows, whose tile holds zeros
  auto load_x = [&](int blk, int kq) {
    const int off = lane * 16 + blk * 4096;
    x[kq][0] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rs_x0, off + kq * 1024, 0, 0));
    if constexpr (NB == 2) x[kq][1] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rs_x1, off + kq * 1024, 0, 0));
  };
  auto product = [&](int st) {
    const int blk0 = step_word(st) >> 2, blk_next = step_word(st + 1) >> 2;
    static_for<0, KB>([&](auto J) {
      constexpr int jb = decltype(J)::value, N = 4 * RT;
      const int after = jb + 1 < KB ? blk0 + jb + 1 : blk_next;  // the block whose X takes the place of this one's
      const uint16_t* const a_even = lds + (st & 1) * TILE + jb * BLOCK + (1 + 8 * mq + (mq & 1)) * kPosPitch + mi * 4;
      const uint16_t* const a_odd = a_even - 2 * (mq & 1) * kPosPitch;
      bf16x8 av[kAhead + 1];
      auto load_a = [&](int n) {
        const int w = n / RT, i = n % RT;
        const u32x2 a0 = *reinterpret_cast<const u32x2*>(a_even + i * kBlockVals + 2 * w * kPosPitch);
        const u32x2 a1 = *reinterpret_cast<const u32x2*>(a_odd + i * kBlockVals + (2 * w + 1) * kPosPitch);
        av[n % (kAhead + 1)] = __builtin_bit_cast(bf16x8, u32x4{a0.x, a0.y, a1.x, a1.y});
      };
#pragma unroll
      for (int n = 0; n < kAhead; ++n) load_a(n);
#pragma unroll
      for (int n = 0; n < N; ++n) {
        if (n + kAhead < N) load_a(n + kAhead);
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
          C[jb][n % RT][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
              av[n % (kAhead + 1)], __builtin_bit_cast(bf16x8, x[n / RT][nb]), C[jb][n % RT][nb], 0, 0, 0);
        if (n % RT == RT - 1) load_x(after, n / RT);
      }
    });
    if ((st + 1) % per_part == 0) {  // KB parts are complete
#pragma unroll
      for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
          f32x4& sum = S[(i * NB + nb) * 64];
          f32x4 t = C[0][i][nb] + C[1][i][nb];
          if (st + 1 > per_part) t = sum + t;
          if constexpr (KB == 4) t += C[2][i][nb] + C[3][i][nb];
          sum = t;
#pragma unroll
          for (int jb = 0; jb < KB; ++jb) C[jb][i][nb] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
    }
  };

  // Step st is decoded between barriers st - 1 and st, multiplied between st and st + 1: by the first four waves behind the
  // decode of step st + 1, by the others, each of which shares a SIMD with one of them, in front of it.  Every wave meets
  // nsteps barriers, one a turn, in front of the product or behind it.
  const int ahead = wv < 4;
  load_mask(0);
  issue(0);
  load_mask(1);
  if (ahead) {
    decode(0);
    __syncthreads();
  }
#pragma unroll
  for (int kq = 0; kq < 4; ++kq) load_x(0, kq);  // behind the windows of a step, as in the loop
  if (!act0) {  // a loop of its own: where loads of X may not have been issued, a wait for the windows waits for X as well
    for (int st = 0; st + 1 < nsteps + !ahead; ++st) {
      decode(st + ahead);
      __syncthreads();
    }
    return;
  }
  for (int st = 0; st < nsteps; ++st) {
    decode(st + ahead);
    if (!ahead) __syncthreads();
    product(st);
    if (ahead && st + 1 < nsteps) __syncthreads();
  }

  // ---- S[i][nb][e]: row 16 i + 4 mq + e, column cb0 + 128 nb + 16 wv + mi
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    const int col = cb0 + 128 * nb + 16 * wv + mi;
    if (col >= a.ncols) continue;
#pragma unroll
    for (int i = 0; i < RT; ++i) {
      const int orow = row0 + 16 * i + 4 * mq;
      const f32x4 s = S[(i * NB + nb) * 64];
      if (a.epi == 0) {
        float* y = a.Y + (size_t)col * a.yld + orow;
        if (orow + 4 <= a.rows) {
          __builtin_memcpy(y, &s, 16);
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (orow + e < a.rows) y[e] = s[e];
        }
      } else if (a.epi == 1) {
        uint16_t* hp = a.out16 + (size_t)col * a.yld + orow;
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (orow + e < a.rows) hp[e] = f32_to_bf16(bf16_to_f32(hp[e]) + round_bf16(s[e]));
      } else {
#pragma unroll
        for (int e = 0; e < 4; e += 2) {
          if (orow + e + 1 < a.rows) {
            const float g = round_bf16(s[e]), u = round_bf16(s[e + 1]);
            a.out16[(size_t)col * (a.yld >> 1) + ((orow + e) >> 1)] = f32_to_bf16(g / (1.0f + expf(-g)) * u);
          }
        }
      }
    }
  }
}

template <int RT>
static size_t wide_lds_bytes(int bw) {
  return sizeof(uint16_t) * 2 * (size_t)(8 * kBlockVals + 64) + wide_pre_bytes<RT>(bw) + sizeof(float) * 16 * RT * kWideCols;
}

// Whether the wide form takes a matrix of this shape: counts of kept values in 16 bits, the LDS (of the smaller form).
static inline bool wide_shape_ok(const cas_ctx* ctx, int64_t rows, int64_t cols, int bw) {
  return rows > 0 && cols < 65536 && wide_lds_bytes<2>(bw) <= (size_t)ctx->lds_max;
}

template <int RT, int NB, bool MX>
static int launch_wide_nb(cas_ctx* ctx, const VerifyArgs& a, int t, int q) {
  const size_t lds = wide_lds_bytes<RT>(a.bw);
  const int64_t groups = (a.rows + 16 * RT - 1) / (16 * RT);
  const int64_t grid = (groups + kXcds - 1) / kXcds * kXcds * ((a.ncols + kWideCols - 1) / kWideCols);
#define CAS_LAUNCH(TV)                                                                                            \
  case TV: {                                                                                                      \
    static LdsLimit lim;                                                                                          \
    const int rc = allow_lds(ctx, (const void*)gemm_prefill_kernel<TV, RT, NB, MX>, lds, lim);                        \
    if (rc != CAS_OK) return rc;                                                                                  \
    hipLaunchKernelGGL((gemm_prefill_kernel<TV, RT, NB, MX>), dim3((unsigned)grid), dim3(kWideThreads), lds, ctx->stream, a, q); \
  } break;
  switch (t) {
    CAS_LAUNCH(0) CAS_LAUNCH(1) CAS_LAUNCH(2) CAS_LAUNCH(3) CAS_LAUNCH(4) CAS_LAUNCH(5) CAS_LAUNCH(6) CAS_LAUNCH(7)
    default: return CAS_EINVAL;
  }
#undef CAS_LAUNCH
  CAS_HIP(ctx, hipGetLastError());
  return CAS_OK;
}

// Up to 128 columns no wave has a second block: the form with two would read the first one's X twice and multiply it twice
// for sums that nobody stores.  A prompt through one layer, us, two blocks / one: 8B shape 48 tokens 380 / 348, 64 390 /
// 354, 128 413 / 366, over shared exponents 64 399 / 359, 128 414 / 368; 70B shape 64 1087 / 975, 128 1146 / 973; hidden 256 (two
// layers) 64 140 / 135.  The last 256 columns of a longer prompt still take two blocks, whatever is left for them: which
// form it is has to be the same for a whole launch (a branch in the kernel makes loads of X conditional, see the loops).
template <int RT, bool MX>
static int launch_wide_rt(cas_ctx* ctx, const VerifyArgs& a, int t, int q) {
  return a.ncols > kWideCols / 2 ? launch_wide_nb<RT, 2, MX>(ctx, a, t, q) : launch_wide_nb<RT, 1, MX>(ctx, a, t, q);
}

// The parts are those the verification GEMM cuts the rows of the WHOLE matrix (a.yld rows) into.  Rows per
// workgroup: 64, or 32 where 64 would leave a third of the CUs or more without a workgroup (or rows of more than some
// 61000 columns leave no room for the sums of 64).  A prompt through one layer, us, by this rule / with 32 rows
// throughout / with 64: 8B shape 64 tokens 355 / 363 / 499, 256 tokens 455 / 468 / 621, 508 tokens 648 / 662 / 780, over shared
// exponents 358 / 378 / 483, 443 / 463 / 625, 658 / 664 / 802; hidden 2048, 508 tokens 271 / 283 / 369.  Not everywhere the
// best: 70B shape 64 tokens 976 / 948 / 1178, 256 tokens 1257 / 1216 / 1506 (896 workgroups of 64 rows are three and a half
// turns of the CUs, 1792 of 32 seven), 300 tokens 1960 / 2056 / 1959; hidden 5120, 508 tokens 949 / 962 / 902.
template <bool MX>
static int launch_wide(cas_ctx* ctx, const VerifyArgs& a, int t) {
  const int q = verify_parts(a.yld, a.cols);
  const int64_t wgs = (int64_t)((a.rows + 63) / 64) * ((a.ncols + kWideCols - 1) / kWideCols);
  if (wgs * 3 < (int64_t)ctx->num_cu * 2 || wide_lds_bytes<4>(a.bw) > (size_t)ctx->lds_max) return launch_wide_rt<2, MX>(ctx, a, t, q);
  return launch_wide_rt<4, MX>(ctx, a, t, q);
}

}  // namespace cas
