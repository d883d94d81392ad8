// Partial attention kernel over one page of the compressed cache and its launcher, compiled
// in two translation units (exact form / draft form); attention.hip explains the algorithm.
#pragma once
#include "cas_device.hpp"
#include "cas_internal.hpp"

namespace cas {

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

struct AttnArgs {
  KvGeom g;
  const uint32_t* spec_pool;
  const uint32_t* verif_pool;
  const int32_t* page_row;  // page table row of the sequence
  int layer, len, nsplit, pages_per_split;
  const uint16_t* Q;
  int ncols, n_q_heads, grp;  // grp = query heads per kv head
  uint32_t grp_inv;           // ceil(2^16 / grp): row / grp = row * grp_inv >> 16 for rows below 256
  const uint16_t* Knew;
  const uint16_t* Vnew;
  int n_new;
  // fused split of the qkv projection (model path): when qkv != null the columns' q, k, v are
  // taken from the fp32 projection output, rounded to bf16 and rotated here, and the k, v of
  // the columns are also written to their in-flight slots for later passes and the commit
  const float* qkv;   // [ncols][ystride]: q heads, k heads, v heads
  int ystride, slot0; // slot0: in-flight slot of column 0 (its position is len + slot0)
  const float* rope;  // [max_pos][64][2] cos, sin
  uint16_t* Kslot;    // writable views of Knew / Vnew
  uint16_t* Vslot;
  float scale;
  float* part;  // [nsplit][n_kv_heads][R][128] outputs, then [n_kv_heads][R][nsplit] pairs (maximum, sum)
  uint16_t* O;
};

// What differs between the sequences of one launch; blockIdx.z picks the sequence.
constexpr int kAttnBatch = 4;
struct AttnSeq {
  const int32_t* page_row;
  int len, nsplit, ncols, n_new, slot0;
  const uint16_t* Q;
  const uint16_t* Knew;
  const uint16_t* Vnew;
  const float* qkv;
  uint16_t* Kslot;
  uint16_t* Vslot;
  float* part;
  uint16_t* O;
};
struct AttnBatch {
  AttnArgs common;  // its per-sequence members are filled in from s[] inside the kernels
  AttnSeq s[kAttnBatch];
};
__device__ __forceinline__ AttnArgs attn_args_of(const AttnBatch& b, int z) {
  AttnArgs a = b.common;
  const AttnSeq& q = b.s[z];
  a.page_row = q.page_row; a.len = q.len; a.nsplit = q.nsplit; a.ncols = q.ncols; a.n_new = q.n_new;
  a.slot0 = q.slot0; a.Q = q.Q; a.Knew = q.Knew; a.Vnew = q.Vnew; a.qkv = q.qkv;
  a.Kslot = q.Kslot; a.Vslot = q.Vslot; a.part = q.part; a.O = q.O;
  return a;
}

constexpr int kPartStride = 132;  // floats of workspace per (split, row): 128 outputs, maximum and sum, 2 to spare

// The columns of one call in runs: blockIdx.z picks a run of run_cols of them (the last may be shorter), which reads
// the positions before it from the cache; every pointer steps on by its columns.  A form of its own, since the steps
// cost the decode pass up to 1.7 % (four sequences of the 8B shape, 9.10 -> 9.25 ms).
constexpr int kAttnRuns = 32;
struct AttnRuns {
  AttnArgs first;  // the members of the first run
  int run_cols, cols;
  uint32_t run_page[kAttnRuns];  // pages of the runs before: where the run's partial results begin
};
__device__ __forceinline__ AttnArgs attn_args_of(const AttnRuns& b, int z) {
  AttnArgs a = b.first;
  const int c0 = z * b.run_cols;
  const size_t qo = (size_t)c0 * a.n_q_heads * 128, ko = (size_t)c0 * a.g.n_kv_heads * 128;
  a.len += c0;
  a.ncols = a.n_new = min(b.run_cols, b.cols - c0);
  a.nsplit = (a.len + a.ncols + 63) >> 6;
  a.Q += qo; a.O += qo; a.Knew += ko; a.Vnew += ko;
  a.part += (size_t)b.run_page[z] * a.n_q_heads * b.run_cols * kPartStride;
  return a;
}
__host__ __device__ inline const AttnArgs& attn_common(const AttnBatch& b) { return b.common; }
__host__ __device__ inline const AttnArgs& attn_common(const AttnRuns& b) { return b.first; }

constexpr int kPT = 64;          // tokens per page
constexpr int kQP = 136;         // Q row pitch (bf16)
// K and V of a wave's 16 tokens in LDS: [1 + 32 positions][64] values, the four words of a token at one position side by
// side for K, the tokens of a word for V (row 0 takes what lanes without a value left write).  At most two lanes of a wave
// meet in a bank, whatever positions they are at; with rows of a token (K) or a channel (V) in order the writes of the
// walks met in banks for half of the cycles in which the LDS was active, and it was active for 78 % of the kernel's
// (draft form, four sequences of up to 32768 positions: 80 us, 76 with this order; the LDS is active for 63 % of the
// kernel's cycles, 37 % of that for the second lane of a bank).
constexpr int kPos = 64;          // values of a position
constexpr int kWaveKV = 33 * kPos;
constexpr int kPP = 72;          // probability row pitch (bf16)
constexpr int kPagesPerSplit = 1;
constexpr int kMaxCols = 16;     // columns of one pass whose k, v may be split from the projection here

// the (maximum, sum) pairs of a sequence: those of a row lie side by side, as the merge reads them
__device__ __forceinline__ float2* attn_ml(const AttnArgs& a, int R) {
  return reinterpret_cast<float2*>(a.part + (size_t)a.nsplit * a.g.n_kv_heads * R * 128);
}

constexpr int kKVTile = 4 * kWaveKV;  // K and V share one region
constexpr int kQPRows = kQP > 2 * kPP ? kQP : 2 * kPP;                  // Q and (P head, P remainder) share one region

template <int MT>
constexpr size_t attn_lds_bytes() {
  return sizeof(uint16_t) * (MT * 16 * kQPRows + kKVTile) + sizeof(float) * (8 * MT * 16);
}

__device__ __forceinline__ uint32_t low_halves(uint32_t x, uint32_t y) { return __builtin_amdgcn_perm(y, x, 0x05040100u); }
__device__ __forceinline__ uint32_t high_halves(uint32_t x, uint32_t y) { return __builtin_amdgcn_perm(y, x, 0x07060302u); }

// where a channel of a query lies in its row in LDS: the four words of a position side by side, as K has them
__device__ __forceinline__ int q_index(int ch) { return (ch & 31) * 4 + (ch >> 5); }
// the channel of value i of a partial result: a wave's 16 columns are four positions of each word
__device__ __forceinline__ int part_channel(int i) { return ((i >> 2) & 3) * 32 + (i >> 5) * 8 + ((i >> 4) & 1) * 4 + (i & 3); }

// All-reduce over the 16 lanes of a DPP row by rotations; every lane ends with the result (of a sum, with the
// result of an order of its own).  The rotation is part of the operation: an addition folds the move of a builtin with no
// old value into itself, a maximum does not (the compiler first makes its operands quiet numbers, two more
// operations), so that one is written out, behind the wait states that a rotation of a fresh result needs.
template <int CTRL>
__device__ __forceinline__ float row_rot(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
__device__ __forceinline__ float row16_max(float v) {
  asm volatile("s_nop 1\n\tv_max_f32_dpp %0, %0, %0 row_ror:1 row_mask:0xf bank_mask:0xf\n\t"
               "s_nop 1\n\tv_max_f32_dpp %0, %0, %0 row_ror:2 row_mask:0xf bank_mask:0xf\n\t"
               "s_nop 1\n\tv_max_f32_dpp %0, %0, %0 row_ror:4 row_mask:0xf bank_mask:0xf\n\t"
               "s_nop 1\n\tv_max_f32_dpp %0, %0, %0 row_ror:8 row_mask:0xf bank_mask:0xf" : "+v"(v));
  return v;
}
__device__ __forceinline__ float row16_sum(float v) {
  v += row_rot<0x121>(v);
  v += row_rot<0x122>(v);
  v += row_rot<0x124>(v);
  return v + row_rot<0x128>(v);
}

// the first E of four values of a lane group's rows
template <int E>
__device__ __forceinline__ void put_rows(float* dst, const float (&v)[4]) {
  if constexpr (E == 4) *reinterpret_cast<float4*>(dst) = make_float4(v[0], v[1], v[2], v[3]);
  else {
#pragma unroll
    for (int e = 0; e < E; ++e) dst[e] = v[e];
  }
}

// MX: the cache is in the shared-exponent form (one exponent per 32-channel block of a vector)
// E: query rows per lane group of a product.  A product has 16 rows, four per group of 16 lanes, and what follows it up to
// the partial results (masks, maxima, exponentials, rounding, sums) is done row by row of a group: few query rows are
// dealt to the groups, query row rr to row 4 (rr / E) + rr % E, so that R <= 4 MT E rows cost E of the four.
// One column of the 8B heads (4 rows) over four sequences of up to 32768 positions 76 -> 70 us, over 8192 positions 12.5
// -> 11.8 (19 % fewer vector instructions).  5 columns (20 rows of 32; partial results and merge) 24.3 -> 23.5 us over
// 8192 positions, 12.0 -> 11.1 over 1000, draft form 21.2 -> 20.7 and 10.9 -> 10.1; 17 to 24 rows of all head shapes,
// either cache, 1 to 5 %.  9 to 12 rows of one tile and 33 to 36 of three have no form of their own (not tried).
template <int MT, int E, bool FULL, int T, bool MX, class BATCH>
__global__ __launch_bounds__(256) void attn_partial_kernel(BATCH batch) {
  const AttnArgs a = attn_args_of(batch, blockIdx.z);
  if ((int)blockIdx.x >= a.nsplit) return;  // a shorter sequence of the launch: uniform for the workgroup
  extern __shared__ uint16_t lds16[];
  uint16_t* Qs = lds16;                       // [MT*16][kQP]; dead once the scores are in registers
  uint16_t* Ph = lds16;                       // [MT*16][kPP] over the Q region
  uint16_t* Pl = Ph + MT * 16 * kPP;          // [MT*16][kPP]
  uint16_t* Kt = lds16 + MT * 16 * kQPRows;   // [4 waves][kWaveKV]
  uint16_t* Vt = Kt;                          // the K tile is dead once the scores are out
  float* wm = reinterpret_cast<float*>(Kt + kKVTile);  // [4 waves][MT*16] row maximum over the wave's 16 tokens
  float* wl = wm + 4 * MT * 16;                        // [4 waves][MT*16] row sum of exponentials

  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  // the column of a query row without a division (some 20 instructions; there were 8 of them per lane)
  auto col_of = [&](int rr) { return (int)((uint32_t)rr * a.grp_inv >> 16); };
  const int pg = blockIdx.x, head = blockIdx.y;  // one page (64 positions) per workgroup
  const int R = a.ncols * a.grp;
  auto row_of = [](int rr) { return E == 4 ? rr : 4 * (rr / E) + rr % E; };  // row of the products, of query row rr
  const KvGeom& g = a.g;
  const int r = tid >> 2, j = tid & 3;           // decode role: token r of the page, word j
  const int mi = lane & 15, mq = lane >> 4;      // MFMA role
  uint16_t* const kcol = Kt + wv * kWaveKV + kPos + (r & 15) * 4 + j;   // position 0 of the thread's token and word
  uint16_t* const vcol = Vt + wv * kWaveKV + kPos + j * 16 + (r & 15);

  const int total = a.len + a.n_new;             // committed + in-flight positions
  const int tok0 = pg * kPT;
  const int pos = tok0 + r;                      // position of this thread's token
  const bool live = pos < a.len;                 // committed: decode from the cache
  const bool fresh = !live && pos < total;       // in flight: uncompressed vector
  const int first = a.len + a.slot0;             // position of column 0 of this pass
  // in flight and produced by this very pass: split from the projection below by all threads
  const bool own_new = a.qkv != nullptr && fresh && pos >= first;
  // the page table is consulted only for pages that hold committed positions: a page of in-flight
  // positions alone needs no pool page yet (and the plain-bf16 form has no pool at all)
  const int page = tok0 < a.len ? min(max(a.page_row[pg], 0), g.n_pages - 1) : 0;

  // the exact form writes all channels of a page of committed tokens; otherwise what is not written has to read as 0
  const bool clear = !FULL || tok0 + kPT > a.len;
  auto clear_tile = [&](uint16_t* t) {  // the wave's own part
#pragma unroll
    for (int k = 0; k < 4; ++k) reinterpret_cast<uint4*>(t + wv * kWaveKV + kPos)[lane + 64 * k] = make_uint4(0, 0, 0, 0);
  };
  // ---- 0. loads that do not depend on the page table entry go out first: the queries and,
  //         in the fused form, the k, v of this pass's columns that fall into this page
  constexpr int NQ = MT * E;
  float x0[NQ], x1[NQ], cc[NQ], sn[NQ];
  uint32_t qraw[MT][4];
  // fused k, v split: thread (column cf of a batch of 8, channel quarter dq) handles channels
  // dq, dq+32 and their rotation partners dq+64, dq+96
  const int cf = tid >> 5, dq = tid & 31;
  float kx[2][4], vx[2][4];
  float2 kcs[2][2];
  bool fnew[2];
#pragma unroll
  for (int cb = 0; cb < 2; ++cb) {
    const int c = cb * 8 + cf, fpos = first + c;
    fnew[cb] = a.qkv != nullptr && c < a.ncols && fpos >= tok0 && fpos < tok0 + kPT;
  }
  if (a.qkv) {
#pragma unroll
    for (int it = 0; it < NQ; ++it) {  // a wave takes a row at a time
      const int rr = wv + 4 * it, d = lane;
      x0[it] = x1[it] = cc[it] = sn[it] = 0.f;
      if (rr < R) {
        const int c = col_of(rr), gi = rr - c * a.grp;
        const float* src = a.qkv + (size_t)c * a.ystride + (size_t)(head * a.grp + gi) * 128;
        const float2 cs = *reinterpret_cast<const float2*>(a.rope + ((size_t)(first + c) * 64 + d) * 2);
        x0[it] = src[d]; x1[it] = src[d + 64]; cc[it] = cs.x; sn[it] = cs.y;
      }
    }
#pragma unroll
    for (int cb = 0; cb < 2; ++cb) {
      if (fnew[cb]) {
        const int c = cb * 8 + cf;
        const float* src = a.qkv + (size_t)c * a.ystride + (size_t)(a.n_q_heads + head) * 128;
        const float* vsrc = src + (size_t)g.n_kv_heads * 128;
        const float* cs = a.rope + (size_t)(first + c) * 128;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          kx[cb][q] = src[dq + 32 * q];
          vx[cb][q] = vsrc[dq + 32 * q];
        }
        kcs[cb][0] = *reinterpret_cast<const float2*>(cs + 2 * dq);
        kcs[cb][1] = *reinterpret_cast<const float2*>(cs + 2 * (dq + 32));
      }
    }
  } else {
#pragma unroll
    for (int it = 0; it < MT; ++it) {  // two positions of the four words
      const int i = tid + it * 256, rr = i >> 4, d = (i & 15) * 2;
#pragma unroll
      for (int w = 0; w < 4; ++w) qraw[it][w] = 0;
      if (rr < R) {
        const int c = col_of(rr), gi = rr - c * a.grp;
        const uint16_t* src = a.Q + ((size_t)c * a.n_q_heads + head * a.grp + gi) * 128 + d;
#pragma unroll
        for (int w = 0; w < 4; ++w) qraw[it][w] = *reinterpret_cast<const uint32_t*>(src + 32 * w);
      }
    }
  }

  // ---- 1. bitmap words of this thread's (token, word) of K and V; the queries are converted
  //         while they are in flight, then the stream windows are requested
  const size_t tk = (((size_t)a.layer * g.n_pages + page) * 2 + 0) * g.n_kv_heads + head;
  const size_t tv = tk + g.n_kv_heads;
  const uint32_t* ks = a.spec_pool + tk * g.tile_spec_words;
  const uint32_t* vs = a.spec_pool + tv * g.tile_spec_words;
  const uint32_t* kvf = a.verif_pool + tk * g.tile_verif_words;
  const uint32_t* vvf = a.verif_pool + tv * g.tile_verif_words;
  const uint32_t mk = live ? ks[r * 4 + j] : 0u;
  const uint32_t mv = live ? vs[r * 4 + j] : 0u;
  int ek = 0, ev = 0;  // shared-exponent form: exponent of this thread's block (byte j of the token's word)
  if constexpr (MX) {
    if (live) {
      ek = (int)((ks[kPT * 4 + r] >> (8 * j)) & 0xFFu);
      ev = (int)((vs[kPT * 4 + r] >> (8 * j)) & 0xFFu);
    }
  }
  // ---- 2. queries to LDS: row rr = column * grp + member.  Rows past R stay as they are: a row of the
  //         products depends on its own query alone, and nothing reads those
  if (a.qkv) {
#pragma unroll
    for (int it = 0; it < NQ; ++it) {
      const int rr = wv + 4 * it, d = lane;
      if (rr >= R) break;
      const float a0 = round_bf16(x0[it]), a1 = round_bf16(x1[it]);
      Qs[row_of(rr) * kQP + q_index(d)] = f32_to_bf16(a0 * cc[it] - a1 * sn[it]);
      Qs[row_of(rr) * kQP + q_index(d + 64)] = f32_to_bf16(a1 * cc[it] + a0 * sn[it]);
    }
  } else {
#pragma unroll
    for (int it = 0; it < MT; ++it) {
      const int i = tid + it * 256, rr = i >> 4, d = (i & 15) * 2;
      const uint32_t* q = qraw[it];
      if (E == 4 || rr < 4 * MT * E)
        *reinterpret_cast<uint4*>(Qs + row_of(rr) * kQP + d * 4) =
            make_uint4(low_halves(q[0], q[1]), low_halves(q[2], q[3]), high_halves(q[0], q[1]), high_halves(q[2], q[3]));
    }
  }
  WordWindows<T, FULL, MX> wk, wvw;
  auto word_prefix = [&](uint32_t m) -> uint32_t {  // kept values of the token before word j
    const int cnt = __popc(m);
    const int b0 = quad_dpp<0x00>(cnt), b1 = quad_dpp<0x55>(cnt), b2 = quad_dpp<0xAA>(cnt);
    return (uint32_t)((j > 0 ? b0 : 0) + (j > 1 ? b1 : 0) + (j > 2 ? b2 : 0));
  };
  // the pools are touched only by workgroups whose page holds committed positions (uniform for the
  // workgroup): such a page has a tile of its own, so the rows of its not yet committed tokens can
  // be read as well (their masks are 0 and the decode never looks at their windows)
  const bool has_live = tok0 < a.len;
  auto load_v = [&]() {
    const uint32_t p = word_prefix(mv);
    if (has_live) wvw.load(p, 32u * j - p, vs + g.spec_off + r * g.sw, vvf + r * g.lw, vvf + kPT * g.lw + r * g.pw);
  };
  {
    const uint32_t p = word_prefix(mk);
    if (has_live) wk.load(p, 32u * j - p, ks + g.spec_off + r * g.sw, kvf + r * g.lw, kvf + kPT * g.lw + r * g.pw);
  }
  // the draft form has registers to spare for both windows; the exact form asks for V later
  if constexpr (!FULL) load_v();

  if (clear) clear_tile(Kt);
  // the tokens of this pass may lie in any wave's part of the tile: cleared before they are written (uniform)
  if (a.qkv != nullptr && first < tok0 + kPT && first + a.ncols > tok0) __syncthreads();
  // k, v of this pass's columns: round, rotate k; k goes straight into its tile row, v waits
  // in registers until the tile region is free; both go to their in-flight slots
  uint16_t fv[2][4];
#pragma unroll
  for (int cb = 0; cb < 2; ++cb) {
    if (fnew[cb]) {
      const int c = cb * 8 + cf, fpos = first + c;
      const int tr = fpos - tok0;
      uint16_t* kdst = Kt + (tr >> 4) * kWaveKV + (1 + dq) * kPos + (tr & 15) * 4;
      const size_t so = ((size_t)(fpos - a.len) * g.n_kv_heads + head) * 128;
#pragma unroll
      for (int h = 0; h < 2; ++h) {  // channel pair (dq + 32h, dq + 32h + 64)
        const float a0 = round_bf16(kx[cb][h]), a1 = round_bf16(kx[cb][h + 2]);
        const uint16_t k0 = f32_to_bf16(a0 * kcs[cb][h].x - a1 * kcs[cb][h].y);
        const uint16_t k1 = f32_to_bf16(a1 * kcs[cb][h].x + a0 * kcs[cb][h].y);
        kdst[h] = k0;
        kdst[h + 2] = k1;
        a.Kslot[so + dq + 32 * h] = k0;
        a.Kslot[so + dq + 32 * h + 64] = k1;
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        fv[cb][q] = f32_to_bf16(vx[cb][q]);
        a.Vslot[so + dq + 32 * q] = fv[cb][q];
      }
    }
  }
  __syncthreads();

  // ---- 3. K tile: this thread's 32 channels of its token
  {
    if (fresh && !own_new) {  // positions 8 j ..+7 of the token's four words
      const uint16_t* src = a.Knew + ((size_t)(pos - a.len) * g.n_kv_heads + head) * 128 + 8 * j;
      uint16_t* dst = kcol - j + 8 * j * kPos;
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        uint2 x[4];
#pragma unroll
        for (int w = 0; w < 4; ++w) x[w] = *reinterpret_cast<const uint2*>(src + 32 * w + 4 * q);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const uint32_t x0 = i < 2 ? x[0].x : x[0].y, x1 = i < 2 ? x[1].x : x[1].y, x2 = i < 2 ? x[2].x : x[2].y,
                         x3 = i < 2 ? x[3].x : x[3].y;
          *reinterpret_cast<uint2*>(dst + (4 * q + i) * kPos) =
              i & 1 ? make_uint2(high_halves(x0, x1), high_halves(x2, x3)) : make_uint2(low_halves(x0, x1), low_halves(x2, x3));
        }
      }
    }
    wk.decode(mk, (FULL && live) ? ~mk : 0u, [&](int bp, uint16_t v) { kcol[bp * kPos] = v; }, ek);
  }
  if constexpr (FULL) load_v();
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  // ---- 4. scores of this wave's 16 tokens against all query rows, kept in registers:
  //         lane (mi, mq) holds token 16 wv + mi of rows mt*16 + 4 mq + e
  float sc[MT][4];
  const int visible = total - a.ncols - tok0;  // last token of the page that column 0 sees
  {
    // product kk: position 4 kk + mq in lane group mq
    const uint16_t* b_base = Kt + wv * kWaveKV + (1 + mq) * kPos + 4 * mi;
    const int t = 16 * wv + mi;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      f32x4 C = {0.f, 0.f, 0.f, 0.f};
      const uint16_t* a_base = Qs + (mt * 16 + mi) * kQP + 4 * mq;
#pragma unroll
      for (int kk = 0; kk < 8; ++kk) {
        bf16x4 av = *reinterpret_cast<const bf16x4*>(a_base + kk * 16);
        bf16x4 bv = *reinterpret_cast<const bf16x4*>(b_base + 4 * kk * kPos);
        C = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(av, bv, C, 0, 0, 0);
      }
      float mx[4];
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const int rr = (mt * 4 + mq) * E + e;
        // column c sees positions 0 .. len + n_new - ncols + c
        sc[mt][e] = t <= visible + col_of(rr) ? C[e] * a.scale : -INFINITY;
        mx[e] = row16_max(sc[mt][e]);
      }
      if (mi == 0) put_rows<E>(wm + wv * (MT * 16) + mt * 16 + 4 * mq, mx);
    }
  }
  __syncthreads();  // every wave is done with Q and K: their regions may be overwritten
  if (clear) clear_tile(Vt);
  // ---- 5. softmax numerators of the page, head + remainder in bf16; row sums per wave
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    float ps[4];
    const f32x4 m0 = *reinterpret_cast<const f32x4*>(wm + mt * 16 + 4 * mq),
                m1 = *reinterpret_cast<const f32x4*>(wm + (MT + mt) * 16 + 4 * mq),
                m2 = *reinterpret_cast<const f32x4*>(wm + (2 * MT + mt) * 16 + 4 * mq),
                m3 = *reinterpret_cast<const f32x4*>(wm + (3 * MT + mt) * 16 + 4 * mq);
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int rr = mt * 16 + 4 * mq + e, t = 16 * wv + mi;  // row of the product
      // at least the lowest finite number: where a row sees nothing of the page, its maximum is -inf as its scores are
      const float mx = fmaxf(fmaxf(fmaxf(m0[e], m1[e]), fmaxf(m2[e], m3[e])), -3.402823466e38f);
      const float p = __expf(sc[mt][e] - mx);
      const uint16_t ph = f32_to_bf16(p);
      Ph[rr * kPP + t] = ph;
      Pl[rr * kPP + t] = f32_to_bf16(p - bf16_to_f32(ph));
      ps[e] = row16_sum(p);
    }
    // lane 0's sums: the lanes of a row add the same values in orders of their own
    if (mi == 0) put_rows<E>(wl + wv * (MT * 16) + mt * 16 + 4 * mq, ps);
  }
  if (clear) __syncthreads();
  // ---- 6. V tile
  {
    if (fresh && !own_new) {
      const uint16_t* src = a.Vnew + ((size_t)(pos - a.len) * g.n_kv_heads + head) * 128 + 32 * j;
#pragma unroll
      for (int c = 0; c < 32; ++c) vcol[c * kPos] = src[c];
    }
#pragma unroll
    for (int cb = 0; cb < 2; ++cb) {
      if (fnew[cb]) {
        const int tr = first + cb * 8 + cf - tok0;
#pragma unroll
        for (int q = 0; q < 4; ++q) Vt[(tr >> 4) * kWaveKV + (1 + dq) * kPos + q * 16 + (tr & 15)] = fv[cb][q];
      }
    }
    wvw.decode(mv, (FULL && live) ? ~mv : 0u, [&](int bp, uint16_t v) { vcol[bp * kPos] = v; }, ev);
  }
  __syncthreads();
  // ---- 7. O = P V; wave w owns positions 8w .. 8w+7 of the four words, column n of a product position n % 4 of word
  //         n / 4 (part_channel); partial result of this page
  float* part = a.part + ((size_t)pg * g.n_kv_heads + head) * R * 128;
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) {
      f32x4 C = {0.f, 0.f, 0.f, 0.f};
      const uint16_t* b_base = Vt + (1 + 8 * wv + 4 * nt + (mi & 3)) * kPos + (mi >> 2) * 16 + 4 * mq;
      const uint16_t* ah = Ph + (mt * 16 + mi) * kPP + 4 * mq;
      const uint16_t* al = Pl + (mt * 16 + mi) * kPP + 4 * mq;
#pragma unroll
      for (int kb = 0; kb < 4; ++kb) {
        bf16x4 bv = *reinterpret_cast<const bf16x4*>(b_base + kb * kWaveKV);
        C = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(*reinterpret_cast<const bf16x4*>(ah + kb * 16), bv, C, 0, 0, 0);
        C = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(*reinterpret_cast<const bf16x4*>(al + kb * 16), bv, C, 0, 0, 0);
      }
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const int rr = (mt * 4 + mq) * E + e;
        if (rr < R) part[rr * 128 + 32 * wv + nt * 16 + mi] = C[e];
      }
    }
  }
  if (tid < R) {
    const float* m4 = wm + row_of(tid);
    const float* l4 = wl + row_of(tid);
    attn_ml(a, R)[((size_t)head * R + tid) * a.nsplit + pg] =
        make_float2(fmaxf(fmaxf(m4[0], m4[MT * 16]), fmaxf(m4[2 * MT * 16], m4[3 * MT * 16])),
                    ((l4[0] + l4[MT * 16]) + l4[2 * MT * 16]) + l4[3 * MT * 16]);
  }
}

template <int MT, int E, bool FULL, bool MX, class BATCH>
int launch_rows(cas_ctx* ctx, const BATCH& a, dim3 grid) {
  constexpr size_t lds = attn_lds_bytes<MT>();
#define CAS_LAUNCH(TV)                                                                                     \
  case TV: {                                                                                               \
    static LdsLimit lim;                                                                                   \
    const int rc = allow_lds(ctx, (const void*)attn_partial_kernel<MT, E, FULL, TV, MX, BATCH>, lds, lim);            \
    if (rc != CAS_OK) return rc;                                                                           \
    hipLaunchKernelGGL((attn_partial_kernel<MT, E, FULL, TV, MX, BATCH>), grid, dim3(256), lds, ctx->stream, a);      \
  } break;
  switch (attn_common(a).g.t) {
    CAS_LAUNCH(0) CAS_LAUNCH(1) CAS_LAUNCH(2) CAS_LAUNCH(3) CAS_LAUNCH(4) CAS_LAUNCH(5) CAS_LAUNCH(6) CAS_LAUNCH(7)
    default: return CAS_EINVAL;
  }
#undef CAS_LAUNCH
  CAS_HIP(ctx, hipGetLastError());
  return CAS_OK;
}

// query rows of a kv head in the widest call of a launch
inline int attn_rows(const AttnRuns& b) { return b.run_cols * b.first.grp; }
inline int attn_rows(const AttnBatch& b) {
  int cols = 0;
  for (const AttnSeq& q : b.s) cols = q.ncols > cols ? q.ncols : cols;
  return cols * b.common.grp;
}

template <int MT, bool FULL, bool MX = false, class BATCH = AttnBatch>
int launch_mt(cas_ctx* ctx, const BATCH& a, dim3 grid) {
  if constexpr (MT == 1) {
    const int rows = attn_rows(a);
    if (rows <= 4) return launch_rows<1, 1, FULL, MX>(ctx, a, grid);
    if (rows <= 8) return launch_rows<1, 2, FULL, MX>(ctx, a, grid);
  }
  if constexpr (MT == 2) {
    if (attn_rows(a) <= 24) return launch_rows<2, 3, FULL, MX>(ctx, a, grid);
  }
  return launch_rows<MT, 4, FULL, MX>(ctx, a, grid);
}

}  // namespace cas
