// Compressed, paged KV cache: online formatting of new K/V vectors (Sec. 5.1 encoder,
// Sec. 4.2 per-token magnitude pruning) and a reference read-back.
//
// A tile holds the vectors of one (layer, page, K-or-V, kv head): page_tokens rows of
// head_dim = 128 values, K kept per row, in the same four-stream layout as a weight matrix
// (bitmap and spec in the speculation pool; lo and pruned in the verification pool).
#include "cas_device.hpp"
#include "cas_internal.hpp"

namespace cas {

// A wave formats four 128-value vectors, the tokens of four rows of a page that follow one another: 16 lanes per vector,
// eight columns per lane.  Four waves take sixteen rows of a tile, from a multiple of sixteen on, so that whole runs of
// lines are written.  The K-th largest magnitude is found bit by bit (15 of them); a lane counts its keys against a
// candidate two to a register (the upper bit of each half of a difference), the lanes of a vector add up through DPP.
// Equals of the K-th are kept in the order of the columns.  Kept values go to a list in LDS by rank, of which a lane packs
// 16 into the 16-T half words that their fields fill; the pruned ones to their place in the row.
// One wave per vector with ballots (kv_append_few_kernel) is bound on a full chip by the scalar unit, which the SIMDs of a CU
// share (298 scalar instructions per vector): 1021 tokens of 8 heads 11.6 us, so 7.7, of which the search takes 2 (5.6 with one step of the
// fifteen, 6.7 with eight: some 19 vector instructions a step and four vectors); the rest is launch, memory and packing.
constexpr int kAppendWaves = 4, kAppendRows = 4 * kAppendWaves;
constexpr int kKeptPitch = 136;  // values of a list of kept ones: 16-byte steps, and vectors four banks apart

// over the 16 lanes of a DPP row: the sum in every lane, and the sum of the lanes before
__device__ __forceinline__ int row16_add(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x121, 0xf, 0xf, true);  // row_ror 1, 2, 4, 8
  v += __builtin_amdgcn_update_dpp(0, v, 0x122, 0xf, 0xf, true);
  v += __builtin_amdgcn_update_dpp(0, v, 0x124, 0xf, 0xf, true);
  return v + __builtin_amdgcn_update_dpp(0, v, 0x128, 0xf, 0xf, true);
}
__device__ __forceinline__ int row16_before(int v) {
  int s = v;
  s += __builtin_amdgcn_update_dpp(0, s, DPP_ROW_SHR1, 0xf, 0xf, false);
  s += __builtin_amdgcn_update_dpp(0, s, DPP_ROW_SHR2, 0xf, 0xf, false);
  s += __builtin_amdgcn_update_dpp(0, s, DPP_ROW_SHR4, 0xf, 0xf, false);
  s += __builtin_amdgcn_update_dpp(0, s, DPP_ROW_SHR8, 0xf, 0xf, false);
  return s - v;
}

struct AppendStage {  // of a wave
  uint16_t kept[4][kKeptPitch];
  uint32_t bitmap[4][4], sexp[4];
  uint32_t spec[4 * 64], lo[4 * 32], pruned[4 * 64];  // rows side by side, as in the tile
};

template <int T, bool MX>
__global__ __launch_bounds__(64 * kAppendWaves) void kv_append_kernel(KvGeom g, uint32_t* spec_pool, uint32_t* verif_pool,
                                                                      const int32_t* __restrict__ page_row, int layer0,
                                                                      int pos0, int n_tok, const uint16_t* __restrict__ Kn,
                                                                      const uint16_t* __restrict__ Vn, size_t layer_stride) {
  constexpr int FW = MX ? 9 - T : 16 - T;
  __shared__ __attribute__((aligned(16))) AppendStage stages[kAppendWaves];
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  AppendStage& st = stages[wv];
  // grid.z = 2 * (layers of this launch): the vectors of layer layer0 + i start i * layer_stride
  // values after those of layer0
  const int head = blockIdx.y, kv = blockIdx.z & 1, layer = layer0 + (blockIdx.z >> 1);
  const int posw = (pos0 & -kAppendRows) + blockIdx.x * kAppendRows + 4 * wv;  // position of the wave's first row
  const int ra = max(pos0 - posw, 0), rb = min(pos0 + n_tok - posw, 4);        // the wave's rows ra .. rb - 1 are new
  if (ra >= rb) return;  // the waves do not wait for each other
  const int page = page_row[posw / 64], row = posw % 64;
  const int q = lane >> 4, l = lane & 15;  // vector of the wave, columns 8 l .. 8 l + 7
  const int tok = posw + min(max(q, ra), rb - 1) - pos0;  // rows that are not new repeat one that is
  const uint16_t* src = (kv ? Vn : Kn) + (size_t)(blockIdx.z >> 1) * layer_stride +
                        ((size_t)tok * g.n_kv_heads + head) * 128 + 8 * l;
  uint32_t w[4];  // columns 2 i and 2 i + 1
  __builtin_memcpy(w, src, 16);

  constexpr uint32_t kTop = 0x80008000u;
  uint32_t key[4];  // magnitudes under a set bit: a candidate of up to 0x8000 taken off either half leaves that bit if it is reached
#pragma unroll
  for (int i = 0; i < 4; ++i) key[i] = w[i] | kTop;
  uint32_t th = 0;  // the K-th largest magnitude, in both halves
#pragma unroll
  for (int bit = 14; bit >= 0; --bit) {
    const uint32_t cand = th | (0x00010001u << bit);
    int n = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) n += __popc((key[i] - cand) & kTop);
    th = row16_add(n) >= g.K ? cand : th;
  }
  // columns of the lane, bit c = column 8 l + c: those that reach the candidate
  auto reach = [&](uint32_t cand) -> uint32_t {
    uint32_t x = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) x |= ((key[i] - cand) & kTop) >> (15 - 2 * i);
    return (x | (x >> 15)) & 0xFFu;
  };
  const uint32_t larger = reach(th + 0x00010001u);
  uint32_t equal = reach(th) & ~larger;
  // the larger ones, and as many of the equals as are needed, in the order of the columns
  const int n_equal = __popc(equal);
  const int need = g.K - row16_add(__popc(larger)) - row16_before(n_equal);  // of this lane's equals and those behind
  uint32_t kept = larger | (need >= n_equal ? equal : 0u);
  if (__builtin_amdgcn_ballot_w64(need > 0 && need < n_equal)) {  // the line falls among the equals of a lane
    int left = need < n_equal ? need : 0;
    for (; __builtin_amdgcn_ballot_w64(left > 0); --left) {
      const uint32_t low = left > 0 ? equal & (0u - equal) : 0u;
      kept |= low;
      equal ^= low;
    }
  }
  const int n_kept = __popc(kept);
  int rank = row16_before(n_kept);

  // shared-exponent form: the exponent of a 32-channel block, four lanes, is the largest among its kept values (0 for a
  // block without any)
  int E = 0;
  if constexpr (MX) {
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      const uint32_t v = (w[c >> 1] >> (16 * (c & 1))) & 0xFFFFu;
      if ((kept >> c) & 1u) E = max(E, eff_exponent(v));
    }
    E = max(E, quad_dpp<0xB1>(E));  // the lane beside, the other pair
    E = max(E, quad_dpp<0x4E>(E));
    if ((l & 3) == 0) reinterpret_cast<uint8_t*>(&st.sexp[q])[l >> 2] = (uint8_t)E;
  }
  reinterpret_cast<uint8_t*>(st.bitmap[q])[l] = (uint8_t)kept;
  uint16_t* const pr = reinterpret_cast<uint16_t*>(st.pruned + q * g.pw);
  uint16_t* const kp = st.kept[q];
  if (g.K + l < kKeptPitch) kp[g.K + l] = 0;  // up to a whole group of 16
  // the upper half of a row's last word may belong to no value
  if (l == 0 && (g.K & 1)) pr[128 - g.K] = 0;
  if (l == 1 && g.sw > 0) st.spec[q * g.sw + g.sw - 1] = 0;
  if (l == 2 && g.lw > 0) st.lo[q * g.lw + g.lw - 1] = 0;
  int gap = 8 * l - rank;  // pruned values before the column
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    const uint32_t v = (w[c >> 1] >> (16 * (c & 1))) & 0xFFFFu;
    const bool k = (kept >> c) & 1u;
    uint32_t u = v;
    if constexpr (MX) {  // sign + magnitude: the significand shifted down to the block's exponent
      const int sh = E - eff_exponent(v);
      u = ((v >> 15) << 8) | (sh < 8 ? significand(v) >> sh : 0u);
    }
    *(k ? kp + rank : pr + gap) = (uint16_t)(MX ? (k ? u : v) : v);
    rank += k;
    gap += !k;
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();

  if (16 * l < g.K) {  // values 16 l .. 16 l + 15 of the kept ones: FW half words of fields, T of dropped bits
    uint32_t v[8];
    *reinterpret_cast<uint4*>(v) = reinterpret_cast<const uint4*>(kp)[2 * l];
    *reinterpret_cast<uint4*>(v + 4) = reinterpret_cast<const uint4*>(kp)[2 * l + 1];
    auto pack = [&](auto W, auto DOWN, uint32_t* out, int words) {
      constexpr int width = decltype(W)::value, down = decltype(DOWN)::value, NW = (width + 1) / 2;
      uint32_t o[NW];
#pragma unroll
      for (int i = 0; i < NW; ++i) o[i] = 0;
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const uint32_t f = __builtin_amdgcn_ubfe(v[i >> 1], 16 * (i & 1) + down, width);
        const int bit = i * width, k = bit >> 5, sh = bit & 31;
        o[k] |= f << sh;
        if (sh + width > 32) o[min(k + 1, NW - 1)] |= f >> (32 - sh);
      }
      if constexpr ((width & 1) == 0) {
#pragma unroll
        for (int i = 0; i < NW; ++i)
          if (l * NW + i < words) out[l * NW + i] = o[i];
      } else {
        uint16_t* const h = reinterpret_cast<uint16_t*>(out) + l * width;
#pragma unroll
        for (int i = 0; i < width; ++i)
          if (l * width + i < 2 * words) h[i] = (uint16_t)(o[i >> 1] >> (16 * (i & 1)));
      }
    };
    pack(std::integral_constant<int, FW>{}, std::integral_constant<int, T>{}, st.spec + q * g.sw, g.sw);
    if constexpr (T > 0) pack(std::integral_constant<int, T>{}, std::integral_constant<int, 0>{}, st.lo + q * g.lw, g.lw);
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();

  if (page < 0 || page >= g.n_pages) return;  // a page table entry outside the pool: nothing is written
  const size_t tile = (((size_t)layer * g.n_pages + page) * 2 + kv) * g.n_kv_heads + head;
  uint32_t* ts = spec_pool + tile * g.tile_spec_words;
  uint32_t* tv = verif_pool + tile * g.tile_verif_words;
  // the new rows of the wave, words of a stream each: read together, then written
  uint32_t vb, ve = 0, vs[4], vl[2], vp[4];
  vb = (&st.bitmap[0][0])[lane & 15];
  if constexpr (MX) ve = st.sexp[lane & 3];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    if (16 * k < g.sw) vs[k] = st.spec[64 * k + lane];
    if (k < 2 && 16 * k < g.lw) vl[k & 1] = st.lo[64 * k + lane];
    if (16 * k < g.pw) vp[k] = st.pruned[64 * k + lane];
  }
  auto flush = [&](uint32_t v, uint32_t* to, int words, int i) {
    if (i >= ra * words && i < rb * words) to[row * words + i] = v;
  };
  flush(vb, ts, 4, lane);
  if constexpr (MX) flush(ve, ts + 256, 1, lane);
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    if (16 * k < g.sw) flush(vs[k], ts + g.spec_off, g.sw, 64 * k + lane);
    if (k < 2 && 16 * k < g.lw) flush(vl[k & 1], tv, g.lw, 64 * k + lane);
    if (16 * k < g.pw) flush(vp[k], tv + 64 * g.lw, g.pw, 64 * k + lane);
  }
}

// One wave per vector, for launches that leave most of the chip idle (see the launch): what counts there is how long one
// wave takes from end to end, and a step of the search is a compare, a ballot and a scalar count here, a chain of some twelve
// dependent vector operations above.  All 15 bits are searched: ending when K values are left costs a branch per bit, as
// much as it saves.  Bound by dependent instructions between two memory round trips; 1.55 of the 2.65 us are the launch.
__global__ __launch_bounds__(64 * kAppendWaves) void kv_append_few_kernel(KvGeom g, uint32_t* spec_pool, uint32_t* verif_pool,
                                                                          const int32_t* __restrict__ page_row, int layer0,
                                                                          int pos0, int n_tok, const uint16_t* __restrict__ Kn,
                                                                          const uint16_t* __restrict__ Vn, size_t layer_stride) {
  __shared__ uint32_t stages[kAppendWaves][3 * 64 + 8];  // sw + lw + pw <= 16*128/32 = 64 words (+ rounding)
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  uint32_t* const stage = stages[wv];
  // grid.z = 2 * (layers of this launch): the vectors of layer layer0 + i start i * layer_stride
  // values after those of layer0
  const int tok = blockIdx.x * kAppendWaves + wv, head = blockIdx.y, kv = blockIdx.z & 1, layer = layer0 + (blockIdx.z >> 1);
  if (tok >= n_tok) return;  // the waves do not wait for each other
  const int pos = pos0 + tok, page_index = pos / g.page_tokens, row = pos - page_index * g.page_tokens;
  const int page = page_row[page_index];
  const uint16_t* src = (kv ? Vn : Kn) + (size_t)(blockIdx.z >> 1) * layer_stride +
                        ((size_t)tok * g.n_kv_heads + head) * 128;
  const uint32_t v0 = src[lane], v1 = src[lane + 64];
  const uint32_t key0 = v0 & 0x7FFFu, key1 = v1 & 0x7FFFu;
  for (int i = lane; i < g.sw + g.lw + g.pw; i += 64) stage[i] = 0;
  uint32_t T = g.K > 0 ? 0u : 0xFFFFFFFFu;  // the K-th largest magnitude
  auto count = [](uint64_t m0, uint64_t m1) { return __popcll(m0) + __popcll(m1); };
#pragma unroll
  for (int bit = 14; bit >= 0; --bit) {
    const uint32_t cand = T | (1u << bit);
    if (count(__builtin_amdgcn_ballot_w64(key0 >= cand), __builtin_amdgcn_ballot_w64(key1 >= cand)) >= g.K) T = cand;
  }
  // the larger ones, and as many of its equals as are needed, in the order of the columns
  uint64_t m01 = __builtin_amdgcn_ballot_w64(key0 > T), m23 = __builtin_amdgcn_ballot_w64(key1 > T);
  const uint64_t eq0 = __builtin_amdgcn_ballot_w64(key0 == T), eq1 = __builtin_amdgcn_ballot_w64(key1 == T);
  const int need = g.K - count(m01, m23), need1 = need - __popcll(eq0);
  auto rank_in = [](uint64_t m) {
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
  };
  const int e0 = rank_in(eq0), e1 = rank_in(eq1);
  const bool k0 = (key0 > T) | ((key0 == T) & (e0 < need)), k1 = (key1 > T) | ((key1 == T) & (e1 < need1));
  m01 = __builtin_amdgcn_ballot_w64(k0);
  m23 = __builtin_amdgcn_ballot_w64(k1);
  const uint32_t r0 = (uint32_t)rank_in(m01), r1 = (uint32_t)(__popcll(m01) + rank_in(m23));

  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  uint32_t* st_spec = stage;
  uint32_t* st_lo = stage + g.sw;
  uint16_t* st_pr = reinterpret_cast<uint16_t*>(st_lo + g.lw);
  const int fw = g.mx ? 9 - g.t : 16 - g.t;
  const uint32_t lomask = (1u << g.t) - 1u;
  // shared-exponent form: the exponent of a 32-channel block is the largest among its kept values
  // (0 for a block without any); lanes 0..31 / 32..63 hold blocks 0 / 1 in v0 and blocks 2 / 3 in v1
  int E0 = 0, E1 = 0;
  if (g.mx) {
    E0 = k0 ? eff_exponent(v0) : 0;
    E1 = k1 ? eff_exponent(v1) : 0;
#pragma unroll
    for (int d = 1; d < 32; d <<= 1) {
      E0 = max(E0, __shfl_xor(E0, d));
      E1 = max(E1, __shfl_xor(E1, d));
    }
  }
  auto put = [&](uint32_t* s, uint32_t bit, uint32_t v, int width) {
    uint32_t w = bit >> 5, sh = bit & 31;
    atomicOr(&s[w], v << sh);
    if (sh + width > 32) atomicOr(&s[w + 1], v >> (32 - sh));
  };
  auto emit = [&](bool kept, uint32_t v, uint32_t rank, uint32_t col, int E) {
    if (kept) {
      if (g.mx) {  // sign + magnitude: the significand shifted down to the block's exponent
        const int sh = E - eff_exponent(v);
        const uint32_t mag = sh < 8 ? significand(v) >> sh : 0u;
        put(st_spec, rank * fw, ((v >> 15) << (8 - g.t)) | (mag >> g.t), fw);
        if (g.t) put(st_lo, rank * g.t, mag & lomask, g.t);
      } else {
        put(st_spec, rank * fw, v >> g.t, fw);
        if (g.t) put(st_lo, rank * g.t, v & lomask, g.t);
      }
    } else {
      st_pr[col - rank] = (uint16_t)v;
    }
  };
  emit(k0, v0, r0, (uint32_t)lane, E0);
  emit(k1, v1, r1, (uint32_t)lane + 64u, E1);
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();

  if (page < 0 || page >= g.n_pages) return;  // a page table entry outside the pool: nothing is written
  const size_t tile = (((size_t)layer * g.n_pages + page) * 2 + kv) * g.n_kv_heads + head;
  uint32_t* ts = spec_pool + tile * g.tile_spec_words;
  uint32_t* tv = verif_pool + tile * g.tile_verif_words;
  if (lane < 4) {
    uint64_t m = lane < 2 ? m01 : m23;
    ts[row * 4 + lane] = (uint32_t)(m >> ((lane & 1) * 32));
  }
  if (g.mx) {  // the four block exponents of the vector, block j in byte j
    const int e01 = __shfl(E0, 0) | (__shfl(E0, 32) << 8), e23 = __shfl(E1, 0) | (__shfl(E1, 32) << 8);
    if (lane == 0) ts[g.page_tokens * 4 + row] = (uint32_t)(e01 | (e23 << 16));
  }
  uint32_t* dspec = ts + g.spec_off + row * g.sw;
  uint32_t* dlo = tv + row * g.lw - g.sw;
  uint32_t* dpr = tv + g.page_tokens * g.lw + row * g.pw - g.sw - g.lw;
  for (int i = lane; i < g.sw + g.lw + g.pw; i += 64) (i < g.sw ? dspec : i < g.sw + g.lw ? dlo : dpr)[i] = stage[i];
}

// Reference read-back of cached vectors to dense bf16 (full == 0: zero-padded draft view).
__global__ __launch_bounds__(128) void kv_read_kernel(KvGeom g, const uint32_t* spec_pool, const uint32_t* verif_pool,
                                                      const int32_t* __restrict__ page_row, int layer, int pos0,
                                                      int full, uint16_t* Ko, uint16_t* Vo) {
  const int col = threadIdx.x;
  const int tok = blockIdx.x, head = blockIdx.y, kv = blockIdx.z;
  const int pos = pos0 + tok;
  int page = page_row[pos / g.page_tokens];
  if (page < 0 || page >= g.n_pages) {  // a page table entry outside the pool reads as zeros
    (kv ? Vo : Ko)[((size_t)tok * g.n_kv_heads + head) * 128 + col] = 0;
    return;
  }
  const int row = pos % g.page_tokens;
  const size_t tile = (((size_t)layer * g.n_pages + page) * 2 + kv) * g.n_kv_heads + head;
  const uint32_t* ts = spec_pool + tile * g.tile_spec_words;
  const uint32_t* tv = verif_pool + tile * g.tile_verif_words;
  const uint32_t* bm = ts + row * 4;
  const int j = col >> 5, c = col & 31;
  uint32_t p = 0;
  for (int i = 0; i < j; ++i) p += __popc(bm[i]);
  const uint32_t m = bm[j];
  p += __popc(m & ((1u << c) - 1u));
  const int fw = g.mx ? 9 - g.t : 16 - g.t;
  uint32_t v;
  if ((m >> c) & 1u) {
    v = read_field(ts + g.spec_off + row * g.sw, p * fw, fw);
    const uint32_t lo = (full && g.t) ? read_field(tv + row * g.lw, p * g.t, g.t) : 0u;
    if (g.mx) {
      const int E = (int)((ts[g.page_tokens * 4 + row] >> (8 * j)) & 0xFFu);
      v = mx_word(v >> (8 - g.t), E, ((v & ((1u << (8 - g.t)) - 1u)) << g.t) | lo);
    } else {
      v = (v << g.t) | lo;
    }
  } else {
    v = full ? read_field(tv + g.page_tokens * g.lw + row * g.pw, ((uint32_t)col - p) * 16, 16) : 0u;
  }
  uint16_t* dst = (kv ? Vo : Ko) + ((size_t)tok * g.n_kv_heads + head) * 128;
  dst[col] = (uint16_t)v;
}

int launch_kv_append(cas_ctx* ctx, cas_kv* kv, int layer, int seq, const uint16_t* K, const uint16_t* V, int n_tok,
                     int pos0) {
  return launch_kv_append_layers(ctx, kv, layer, 1, 0, seq, K, V, n_tok, pos0);
}

int launch_kv_append_layers(cas_ctx* ctx, cas_kv* kv, int layer0, int n_layers, size_t layer_stride, int seq,
                            const uint16_t* K, const uint16_t* V, int n_tok, int pos0) {
  if (n_tok <= 0 || n_layers <= 0) return CAS_OK;
  const KvGeom& g = kv->geom;
  // Up to twelve vectors per CU (ten over shared exponents) a wave takes each, above four.  us, one wave a vector / a wave
  // for four, 600 per mille kept, t = 4: 1 token of 8 heads 2.65 / 3.63, 64 of 8 (1024 vectors) 2.98 / 3.92, 2048 vectors 3.33 /
  // 3.99, 3072 4.02 / 4.02, 4000 4.61 / 4.06, 8192 6.83 / 5.55; over shared exponents 2.94 / 3.79, 3.30 / 4.00, 3.72 / 4.11, 3072
  // 4.33 / 4.14, 4000 4.99 / 4.17.  A commit of 5 positions of 8 layers, event to event, 6.1 / 7.1, of 80 layers (6400) 11.1 / 9.0.
  if ((int64_t)n_tok * g.n_kv_heads * 2 * n_layers <= (int64_t)(g.mx ? 10 : 12) * ctx->num_cu) {
    const dim3 grid((n_tok + kAppendWaves - 1) / kAppendWaves, g.n_kv_heads, 2 * n_layers);
    hipLaunchKernelGGL(kv_append_few_kernel, grid, dim3(64 * kAppendWaves), 0, ctx->stream, g, (uint32_t*)kv->d_spec,
                       (uint32_t*)kv->d_verif, kv->d_page_table + (size_t)seq * g.max_pages_per_seq, layer0, pos0, n_tok,
                       K, V, layer_stride);
    CAS_HIP(ctx, hipGetLastError());
    return CAS_OK;
  }
  const int blocks = (pos0 + n_tok - 1) / kAppendRows - pos0 / kAppendRows + 1;
  const dim3 grid(blocks, g.n_kv_heads, 2 * n_layers);
#define CAS_LAUNCH(TV)                                                                                              \
  case TV:                                                                                                          \
    hipLaunchKernelGGL(g.mx ? (kv_append_kernel<TV, true>) : (kv_append_kernel<TV, false>), grid,                   \
                       dim3(64 * kAppendWaves), 0, ctx->stream, g, (uint32_t*)kv->d_spec, (uint32_t*)kv->d_verif,   \
                       kv->d_page_table + (size_t)seq * g.max_pages_per_seq, layer0, pos0, n_tok, K, V, layer_stride); \
    break;
  switch (g.t) {
    CAS_LAUNCH(0) CAS_LAUNCH(1) CAS_LAUNCH(2) CAS_LAUNCH(3) CAS_LAUNCH(4) CAS_LAUNCH(5) CAS_LAUNCH(6) CAS_LAUNCH(7)
    default: return CAS_EINVAL;
  }
#undef CAS_LAUNCH
  CAS_HIP(ctx, hipGetLastError());
  return CAS_OK;
}

int launch_kv_read(cas_ctx* ctx, cas_kv* kv, int layer, int seq, int pos0, int n_tok, int full, uint16_t* K,
                   uint16_t* V) {
  if (n_tok <= 0) return CAS_OK;
  const KvGeom& g = kv->geom;
  dim3 grid(n_tok, g.n_kv_heads, 2);
  hipLaunchKernelGGL(kv_read_kernel, grid, dim3(128), 0, ctx->stream, g, (const uint32_t*)kv->d_spec,
                     (const uint32_t*)kv->d_verif, kv->d_page_table + (size_t)seq * g.max_pages_per_seq, layer, pos0,
                     full, K, V);
  CAS_HIP(ctx, hipGetLastError());
  return CAS_OK;
}

}  // namespace cas
