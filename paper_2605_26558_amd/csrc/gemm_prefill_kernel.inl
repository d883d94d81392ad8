// Kernel template and launcher of the wide verification GEMM: the product of the exact matrix with the
// columns of a long prompt.  The verification GEMM decodes the matrix once per 32 columns at most; here a
// workgroup decodes 16 RT rows once for 256 columns.  Every output has the bits of the verification GEMM:
// the parts a row's columns are cut into, the order of the 16-column products within a part and the order
// in which the parts are added are the same.
#pragma once
#include <algorithm>
#include "gemm_verify_kernel.inl"

namespace cas {

constexpr int kWideThreads = 512;
constexpr int kWideCols = 256;  // columns of X per workgroup

// One workgroup per CU (8 waves of up to 256 registers).  A step takes KB blocks of 128 columns: thread
// (row r, block, word j) places its 32 values in a tile in LDS, each wave multiplies all rows of the tile
// with its own columns n and n + 128 of X, which it reads from memory (no other wave of the workgroup needs
// them).  Two tiles: while one is multiplied the next one is filled, with one barrier per step; the waves
// w and w + 4, which share a SIMD, take the two halves of a step in opposite order, so that the decode of
// the one runs under the matrix operations of the other.  Blocks come part by part (part p of
// Q has the blocks p, p + Q, ...), which makes a part one running sum; the counts of kept values in front of every block of
// every row are made at the start (pre).
// Bound by waiting, not by one unit.  Counters of 28672 x 4096 with 508 columns (386 us): of the 702 K cycles
// that a CU is busy, the matrix operations (8 K flops in 16 cycles) take 229 K on each SIMD and the other
// vector instructions, the decode's 14 or so per value and 256 columns above all, 175 K, 58 % together; LDS is active
// for 177 K (a quarter of it conflicts); each of the two waves of a SIMD waits for 41 % of its cycles (one barrier per
// step, operands from memory).  The CUs are busy for 85 % of the launch (896 workgroups, one per CU at a time).
// With nothing else on the chip the 16x16x16 operations reach 668 TFLOP/s from two waves per SIMD (30 cycles
// an operation at 2.4 GHz) and 736 from eight (17 cycles, but the clock falls to 1.5 GHz under that load).
template <int T, int RT, bool MX>
__global__ __launch_bounds__(kWideThreads) void gemm_prefill_kernel(VerifyArgs a, int Q) {
  constexpr int ROWS = 16 * RT, KB = 128 / ROWS;
  static_assert(KB == 2 || KB == 4, "the fragments of X alternate between two sets");
  constexpr int TILE = KB * RT * kBlockVals;  // values of one tile: blocks of 16 rows x 128 columns
  extern __shared__ uint16_t lds[];
  uint16_t* pre = lds + 2 * TILE;  // [ROWS][nblk] kept values of the row before each block of 128 columns
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ncb = (a.ncols + kWideCols - 1) / kWideCols;
  const int cb0 = (int)(blockIdx.x % ncb) * kWideCols, row0 = (int)(blockIdx.x / ncb) * ROWS;
  const int nblk = (a.bw + 3) >> 2;
  const int per_part = (nblk + Q - 1) / Q;  // blocks of a part: part p has the blocks p, p + Q, ...
  const int nsteps = (Q * per_part + KB - 1) / KB;

  // ---- kept values in front of every block
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
        const int blk = (w0 + lane) >> 2;
        if ((lane & 3) == 0 && blk < nblk) pre[(wv * RW + i) * nblk + blk] = (uint16_t)(run[i] + (uint32_t)(incl - cnt));
        run[i] += (uint32_t)__builtin_amdgcn_readlane(incl, 63);
      }
    }
    __syncthreads();
  }

  // first bitmap word of block b in the order of the sums (b / per_part by multiplication: b per_part <= 2^16
  // for every b before the last step's end); blocks past the end of the rows lie past their words
  const int inv_per = (65536 + per_part - 1) / per_part;
  auto block_word = [&](int b) -> int {
    const int part = b * inv_per >> 16;
    return 4 * ((b - part * per_part) * Q + part);
  };

  // ---- decode role: row r of the tile, block qb of the step (the same for a whole wave), word j of the block
  const int r = (tid >> 2) & (ROWS - 1), qb = wv * 16 / ROWS, j = lane & 3;
  const int row = min(row0 + r, a.rows - 1);
  auto rsrc = [&](const uint32_t* base, int words) {
    return __builtin_amdgcn_make_buffer_rsrc((void*)(base + (size_t)row0 * words), 0, ROWS * 4 * words + 128, kRawBufferFlags);
  };
  const __amdgpu_buffer_rsrc_t rs_s = rsrc(a.spec, a.sw), rs_l = rsrc(a.lo, a.lw), rs_p = rsrc(a.pruned, a.pw);
  const __amdgpu_buffer_rsrc_t rs_b = rsrc(a.bitmap, a.bw);
  const int rr = row - row0, row_s = rr * a.sw * 4, row_l = rr * a.lw * 4, row_p = rr * a.pw * 4, row_b = rr * a.bw * 4;
  uint16_t* const trow = lds + (qb * RT + (r >> 4)) * kBlockVals + kPosPitch + (r & 15) * 4 + j;
  WordWindows<T, true, MX> ww;
  uint32_t m_next = 0, m_cur = 0;
  int e_next = 0, e_cur = 0, nvalid = 0;
  // Loads are issued on every path, past the last step for that step again: where a load may or may not
  // have been issued, the compiler's wait for an older one waits for it as well.
  auto load_mask = [&](int st) {
    const int w = block_word(min(st, nsteps - 1) * KB + qb) + j, wc = min(w, a.bw - 1);
    const uint32_t m = __builtin_amdgcn_raw_buffer_load_b32(rs_b, row_b + wc * 4, 0, 0);
    m_next = w < a.bw ? m : 0u;
    if constexpr (MX) e_next = (int)a.sexp[(size_t)row * a.ew + wc];
  };
  auto issue = [&](int st) {  // windows of the step whose mask came last
    const int w0 = block_word(min(st, nsteps - 1) * KB + qb);
    m_cur = m_next;
    e_cur = e_next;
    const int cnt = __popc(m_cur);
    const int b0 = quad_dpp<0x00>(cnt), b1 = quad_dpp<0x55>(cnt), b2 = quad_dpp<0xAA>(cnt);
    nvalid = a.cols - (w0 + j) * 32;
    // words past the end of the row have no fields: keep their (unused) windows in range
    const uint32_t p = nvalid > 0 ? pre[r * nblk + (w0 >> 2)] + (uint32_t)((j > 0 ? b0 : 0) + (j > 1 ? b1 : 0) + (j > 2 ? b2 : 0)) : 0u;
    ww.k.load(p, rs_s, row_s, rs_l, row_l);
    ww.pr.load(nvalid > 0 ? (uint32_t)(w0 + j) * 32u - p : 0u, rs_p, row_p);
  };
  auto decode = [&](int st) {
    if (st >= nsteps) return;
    uint16_t* dst = trow + (st & 1) * TILE;
    const uint32_t valid = nvalid >= 32 ? 0xFFFFFFFFu : (nvalid <= 0 ? 0u : ((1u << nvalid) - 1u));
    if (nvalid < 32) {  // columns past the end are not placed below
#pragma unroll
      for (int q = 0; q < 32; ++q) dst[q * kPosPitch] = 0;
    }
    ww.decode(m_cur, ~m_cur & valid, [&](int pos, uint16_t v) { dst[pos * kPosPitch] = v; }, MX ? e_cur : 0);
    issue(st + 1);
    load_mask(st + 2);
  };

  // ---- product role: columns cb0 + 16 wv + mi and 128 further; A[i = lane%16][k = 4*(lane/16)..+3]
  const int mi = lane & 15, mq = lane >> 4;
  const bool act0 = cb0 + 16 * wv < a.ncols, act1 = cb0 + 128 + 16 * wv < a.ncols;
  // X comes packed (pack_x_kernel): the fragments of 16 columns and 32 values of k are one run of 1 KB
  const size_t xrow = (size_t)nblk * 4 * 512;  // values of a block of 16 columns
  const uint16_t* const xp0 = a.X + (size_t)((cb0 >> 4) + (act0 ? wv : 0)) * xrow + lane * 8;
  const uint16_t* const xp1 = act1 ? xp0 + 8 * xrow : xp0;
  f32x4 C[RT][2], S[RT][2];  // running sum of the part, sum of the parts before it
#pragma unroll
  for (int i = 0; i < RT; ++i)
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) C[i][nb] = S[i][nb] = f32x4{0.f, 0.f, 0.f, 0.f};
  uint4 xa[4][2], xb[4][2];
  auto load_x = [&](int b, uint4 (&x)[4][2]) {
    const int blk = min(block_word(min(b, nsteps * KB - 1)) >> 2, nblk - 1);  // not used past the end
#pragma unroll
    for (int kq = 0; kq < 4; ++kq) {
      x[kq][0] = *reinterpret_cast<const uint4*>(xp0 + (size_t)(blk * 4 + kq) * 512);
      x[kq][1] = *reinterpret_cast<const uint4*>(xp1 + (size_t)(blk * 4 + kq) * 512);
    }
  };
  auto flush = [&]() {  // the part is complete
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
      for (int nb = 0; nb < 2; ++nb) {
        S[i][nb] += C[i][nb];
        C[i][nb] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
  };
  auto product = [&](int st) {
    if (!act0) return;
    static_for<0, KB>([&](auto J) {
      constexpr int jb = decltype(J)::value;
      const int b = st * KB + jb;
      uint4 (&x)[4][2] = (jb & 1) ? xb : xa;
      load_x(b + 1, (jb & 1) ? xa : xb);
      if (b > per_part - 1 && b % per_part == 0) {
        if (b == per_part) {
#pragma unroll
          for (int i = 0; i < RT; ++i)
#pragma unroll
            for (int nb = 0; nb < 2; ++nb) {
              S[i][nb] = C[i][nb];
              C[i][nb] = f32x4{0.f, 0.f, 0.f, 0.f};
            }
        } else {
          flush();
        }
      }
      if (block_word(b) >= a.bw) return;  // past the end of the rows
      const uint16_t* const a_even = lds + (st & 1) * TILE + jb * RT * kBlockVals + (1 + 8 * mq + (mq & 1)) * kPosPitch + mi * 4;
      const uint16_t* const a_odd = a_even - 2 * (mq & 1) * kPosPitch;
      auto block = [&](auto NB) {
        // Fragments of the rows, half of them one product ahead: with all of them ahead the form of 64 rows, which holds
        // 64 registers of sums, as many of X and 48 of windows, spilled up to 48 (508 tokens through 4 layers 3.97
        // ms, 3.90 so; none of them ahead 3.91)
        bf16x4 av[2][RT];
        auto load_a = [&](int kk, int i) {
          av[kk & 1][i] = *reinterpret_cast<const bf16x4*>((kk & 1 ? a_odd : a_even) + i * kBlockVals + kk * kPosPitch);
        };
#pragma unroll
        for (int i = 0; i < RT; ++i) load_a(0, i);
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) {
#pragma unroll
          for (int i = 0; i < RT; ++i) {
            if (i < RT / 2 && kk < 7) load_a(kk + 1, i);
            if (i >= RT / 2 && kk > 0) load_a(kk, i);
          }
#pragma unroll
          for (int nb = 0; nb < decltype(NB)::value; ++nb) {
            const uint4& f = x[kk >> 1][nb];
            const bf16x4 bv = __builtin_bit_cast(bf16x4, (kk & 1) ? u32x2{f.z, f.w} : u32x2{f.x, f.y});
#pragma unroll
            for (int i = 0; i < RT; ++i)
              C[i][nb] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(av[kk & 1][i], bv, C[i][nb], 0, 0, 0);
          }
        }
      };
      if (act1) block(std::integral_constant<int, 2>{});
      else block(std::integral_constant<int, 1>{});
    });
  };

  load_mask(0);
  load_x(0, xa);
  issue(0);
  load_mask(1);
  decode(0);
  __syncthreads();
  const bool product_first = (wv & 4) != 0;
  for (int st = 0; st < nsteps; ++st) {
    if (product_first) product(st);
    decode(st + 1);
    if (!product_first) product(st);
    __syncthreads();
  }
  if (!act0) return;
  flush();

  // ---- S[i][nb][e]: row 16 i + 4 mq + e, column cb0 + 128 nb + 16 wv + mi
#pragma unroll
  for (int nb = 0; nb < 2; ++nb) {
    const int col = cb0 + 128 * nb + 16 * wv + mi;
    if (col >= a.ncols) continue;
#pragma unroll
    for (int i = 0; i < RT; ++i) {
      const int orow = row0 + 16 * i + 4 * mq;
      const f32x4 s = S[i][nb];
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
  return sizeof(uint16_t) * (2 * (size_t)8 * kBlockVals + (size_t)16 * RT * ((bw + 3) / 4));
}

// Whether the wide form takes a matrix of this shape: counts of kept values in 16 bits, the LDS.
static inline bool wide_shape_ok(const cas_ctx* ctx, int64_t rows, int64_t cols, int bw) {
  return rows > 0 && cols < 65536 && wide_lds_bytes<4>(bw) <= (size_t)ctx->lds_max;
}

template <int RT, bool MX>
static int launch_wide_rt(cas_ctx* ctx, const VerifyArgs& a, int t, int q) {
  const size_t lds = wide_lds_bytes<RT>(a.bw);
  const int64_t grid = (int64_t)((a.rows + 16 * RT - 1) / (16 * RT)) * ((a.ncols + kWideCols - 1) / kWideCols);
#define CAS_LAUNCH(TV)                                                                                            \
  case TV: {                                                                                                      \
    static LdsLimit lim;                                                                                          \
    const int rc = allow_lds(ctx, (const void*)gemm_prefill_kernel<TV, RT, MX>, lds, lim);                        \
    if (rc != CAS_OK) return rc;                                                                                  \
    hipLaunchKernelGGL((gemm_prefill_kernel<TV, RT, MX>), dim3((unsigned)grid), dim3(kWideThreads), lds, ctx->stream, a, q); \
  } break;
  switch (t) {
    CAS_LAUNCH(0) CAS_LAUNCH(1) CAS_LAUNCH(2) CAS_LAUNCH(3) CAS_LAUNCH(4) CAS_LAUNCH(5) CAS_LAUNCH(6) CAS_LAUNCH(7)
    default: return CAS_EINVAL;
  }
#undef CAS_LAUNCH
  CAS_HIP(ctx, hipGetLastError());
  return CAS_OK;
}

// The parts are those the verification GEMM cuts the rows of the WHOLE matrix (a.yld rows) into.  Rows per
// workgroup: 64, or 32 where 64 would leave a third of the CUs or more without a workgroup.  A prompt through one
// layer, us, by this rule / with 32 rows throughout / with 64: 8B shape 65 tokens 466 / 482 / 633, 257 tokens
// 717 / 746 / 825, 513 tokens 940 / 975 / 1070; 70B shape 65 tokens 1335 / 1315 / 1574, 257 tokens 2249 / 2674 /
// 2244, 513 tokens 3784 / 4268 / 4007.
template <bool MX>
static int launch_wide(cas_ctx* ctx, const VerifyArgs& a, int t) {
  const int q = verify_parts(a.yld, a.cols);
  const int64_t wgs = (int64_t)((a.rows + 63) / 64) * ((a.ncols + kWideCols - 1) / kWideCols);
  if (wgs * 3 < (int64_t)ctx->num_cu * 2) return launch_wide_rt<2, MX>(ctx, a, t, q);
  return launch_wide_rt<4, MX>(ctx, a, t, q);
}

}  // namespace cas
