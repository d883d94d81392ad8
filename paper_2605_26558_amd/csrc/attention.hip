// Attention of the decode step over the compressed, paged KV cache (Fig. 2_1 structure;
// Sec. 4.1 decides which data a pass may read): the draft pass rebuilds K and V from the
// speculation data with zero padding, the verification pass rebuilds them exactly from both
// pools.  The vectors of the in-flight tokens (draft tokens not yet verified, or the k+1
// columns of the verification pass) arrive uncompressed and are placed at the page rows their
// positions will occupy, and a split always covers the same fixed number of pages: the value
// of a query therefore depends only on the tokens it sees, not on whether they are already
// committed, nor on the number of columns or the total length.
//
// One workgroup handles one kv head and one page (64 positions) of the sequence:
//   1. thread (token r, word j) decodes its 32 channels of K into a bf16 tile in LDS, ordered by the position in the
//      word so that no more than two of the scattered writes of a wave meet in a bank;
//   2. each wave multiplies its 16 tokens with the query rows (grouped-query: the query heads
//      of the group x columns share the kv head) by 16x16x16 bf16 MFMA; the scaled, masked
//      scores stay in the MFMA result registers;
//   3. softmax numerators of the page per query row: the row maximum and sum go through DPP
//      rotations inside a wave and a few LDS words across the four waves (kept for the
//      merge); probabilities are split into a bf16 head and a bf16 remainder, so the second
//      product keeps 16 mantissa bits, and stored over the query tile, which is dead by then;
//   4. the V tile is decoded over the dead K tile, the tokens of a word and position side by side, and P V is formed
//      in fp32 MFMA registers.
// Partial (max, sum, output) of every page go to the workspace; a merge kernel combines them
// in a fixed order.
#include <algorithm>
#include <atomic>
#include "attention_kernel.inl"

namespace cas {

// the draft form (speculation data only) is compiled in attention_draft.hip
extern template int launch_mt<1, false, false>(cas_ctx*, const AttnBatch&, dim3);
extern template int launch_mt<2, false, false>(cas_ctx*, const AttnBatch&, dim3);
extern template int launch_mt<3, false, false>(cas_ctx*, const AttnBatch&, dim3);
// the forms over a cache with shared exponents: attention_mx.hip, attention_mx_draft.hip
extern template int launch_mt<1, true, true>(cas_ctx*, const AttnBatch&, dim3);
extern template int launch_mt<2, true, true>(cas_ctx*, const AttnBatch&, dim3);
extern template int launch_mt<3, true, true>(cas_ctx*, const AttnBatch&, dim3);
extern template int launch_mt<4, true, true>(cas_ctx*, const AttnBatch&, dim3);
extern template int launch_mt<5, true, true>(cas_ctx*, const AttnBatch&, dim3);
extern template int launch_mt<1, false, true>(cas_ctx*, const AttnBatch&, dim3);
extern template int launch_mt<2, false, true>(cas_ctx*, const AttnBatch&, dim3);
extern template int launch_mt<3, false, true>(cas_ctx*, const AttnBatch&, dim3);

// runs of columns (exact form): attention_runs.hip, attention_mx_runs.hip
extern template int launch_mt<1, true, false>(cas_ctx*, const AttnRuns&, dim3);
extern template int launch_mt<2, true, false>(cas_ctx*, const AttnRuns&, dim3);
extern template int launch_mt<3, true, false>(cas_ctx*, const AttnRuns&, dim3);
extern template int launch_mt<4, true, false>(cas_ctx*, const AttnRuns&, dim3);
extern template int launch_mt<1, true, true>(cas_ctx*, const AttnRuns&, dim3);
extern template int launch_mt<2, true, true>(cas_ctx*, const AttnRuns&, dim3);
extern template int launch_mt<3, true, true>(cas_ctx*, const AttnRuns&, dim3);
extern template int launch_mt<4, true, true>(cas_ctx*, const AttnRuns&, dim3);
extern template int launch_mt<5, true, true>(cas_ctx*, const AttnRuns&, dim3);

// Combine the splits: o = sum_s e^{m_s - M} O_s / sum_s e^{m_s - M} l_s, rounded to bf16.  Splits p, p + 8, ... are
// added one after the other in each of eight parts p, then the parts in order.  The denominator: lane i of part p adds
// splits 64 p + i, 64 p + i + 512, ..., the lanes of a part are added in the order of wave_sum, then the parts in order.
// These orders are fixed: the result depends neither on timing, nor on how many rows ride along, nor on which of the
// two kernels below combines a row.
constexpr int kMergeParts = 8;

__device__ __forceinline__ float split_weight(float m, float M) { return m == -INFINITY ? 0.f : __expf(m - M); }

// One workgroup per (query row, kv head, half of the channels), a wave per part.  Bound by latency: everything a wave
// needs first is requested at once, kMergePre outputs of its part, the maxima of these splits (lane q: the q-th) and
// the pairs of its block of the denominator.  The outputs come through buffer descriptors, of no length past the end
// of the part: what lies there reads as 0 and adds nothing, without a branch per load (with branches the compiler's
// code took 5.2 us where this takes 4.8, and 15.8 for 9.8).
constexpr int kMergePre = 32;
template <class BATCH>
__global__ __launch_bounds__(512, 4) void attn_merge_kernel(BATCH batch) {
  const AttnArgs a = attn_args_of(batch, blockIdx.z >> 1);  // blockIdx.z = 2 * sequence + channel half
  __shared__ float red[2][kMergeParts];
  __shared__ float ps[kMergeParts][64];
  const int rr = blockIdx.x, head = blockIdx.y, lane = threadIdx.x & 63;
  const int part = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int d = (blockIdx.z & 1) * 64 + lane;
  const int R = a.ncols * a.grp, n = a.nsplit;
  if (rr >= R) return;  // a sequence with fewer rows than the widest of the launch
  const size_t step = (size_t)a.g.n_kv_heads * R * 128 * kMergeParts * 4;  // bytes from a split of the part to the next
  const char* base = reinterpret_cast<const char*>(a.part + (((size_t)part * a.g.n_kv_heads + head) * R + rr) * 128);
  const float2* ml = attn_ml(a, R) + ((size_t)head * R + rr) * n;
  const int cnt = (n - part + kMergeParts - 1) / kMergeParts;  // splits of this part
  const int s0 = 64 * part + lane;
  float2 blk = make_float2(-INFINITY, 0.f);
  if (s0 < n) blk = ml[s0];
  float m_own = -INFINITY;
  if (lane < cnt) m_own = ml[part + kMergeParts * lane].x;
  float o[kMergePre];
  auto request = [&](int from) {  // outputs from .. from + kMergePre - 1 of the part
    const int q0 = __builtin_amdgcn_readfirstlane(from);  // uniform, and known to be
    const char* row = base + (size_t)q0 * step;
#pragma unroll
    for (int q = 0; q < kMergePre; ++q) {
      const __amdgpu_buffer_rsrc_t rs =
          __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(row), 0, q0 + q < cnt ? 512 : 0, kRawBufferFlags);
      o[q] = __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, 4 * d, 0, 0));
      row += step;
    }
  };
  request(0);
  float M = blk.x;
  for (int s = s0 + 512; s < n; s += 512) M = fmaxf(M, ml[s].x);
  M = wave_max(M);
  if (lane == 0) red[0][part] = M;
  __syncthreads();
#pragma unroll
  for (int q = 0; q < kMergeParts; ++q) M = fmaxf(M, red[0][q]);
  float den = split_weight(blk.x, M) * blk.y;
  for (int s = s0 + 512; s < n; s += 512) den += split_weight(ml[s].x, M) * ml[s].y;
  den = wave_sum(den);
  if (lane == 0) red[1][part] = den;
  float num = 0.f;
  for (int q0 = 0; q0 < cnt;) {
    const int w = __float_as_int(split_weight(m_own, M));
#pragma unroll
    for (int i = 0; i < kMergePre; ++i) num += __int_as_float(__builtin_amdgcn_readlane(w, i)) * o[i];
    q0 += kMergePre;
    if (q0 >= cnt) break;
    m_own = q0 + lane < cnt ? ml[part + kMergeParts * (q0 + lane)].x : -INFINITY;
    request(q0);
  }
  ps[part][lane] = num;
  __syncthreads();
  if (part == 0) {
    den = 0.f;
#pragma unroll
    for (int q = 0; q < kMergeParts; ++q) den += red[1][q];
#pragma unroll
    for (int q = 1; q < kMergeParts; ++q) num += ps[q][lane];
    const int c = rr / a.grp, gi = rr - c * a.grp;
    a.O[((size_t)c * a.n_q_heads + head * a.grp + gi) * 128 + part_channel(d)] = f32_to_bf16(num / den);
  }
}

// Few splits: a wave per (query row, kv head) with all channels and all parts, no LDS and no barrier: with 4 splits
// 2.8 us for 3.5 of the other, with up to 8 splits of 64 rows of four sequences 4.6 us for 10.7.  One wave's loads
// reach to 32 splits; from there on the other form, whose eight waves share them: 129 splits 4.8 us (4.9 with the
// pairs behind each output, LDS weights and a barrier more), 65 to 513 splits of four sequences 9.8 (13.1).
// A whole attention call of the 8B heads with this form / the other, us: 1 column over 8 pages 8.5 / 9.3, 16 pages 8.8 /
// 9.3, 24 pages 9.0 / 9.4, 32 pages 9.4 / 9.4; 5 columns 11.0 / 12.7, 11.3 / 12.9, 11.8 / 13.2, 12.3 / 13.4; 9 columns
// 12.1 / 14.8, 12.6 / 15.4, 13.7 / 15.8, 14.6 / 16.3.  4 query and 2 kv heads over 32 pages: 9.2 / 9.1 and 10.6 / 10.5.
constexpr int kMergeFew = 32;
template <class BATCH>
__global__ __launch_bounds__(256) void attn_merge_few_kernel(BATCH batch) {
  const AttnArgs a = attn_args_of(batch, blockIdx.z);
  const int rr = 4 * blockIdx.x + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), head = blockIdx.y, lane = threadIdx.x & 63;
  const int R = a.ncols * a.grp, n = a.nsplit;
  if (rr >= R) return;
  const size_t sstride = (size_t)a.g.n_kv_heads * R * 64;
  const float2* base = reinterpret_cast<const float2*>(a.part) + ((size_t)head * R + rr) * 64 + lane;
  float2 ml = make_float2(-INFINITY, 0.f);
  if (lane < n) ml = attn_ml(a, R)[((size_t)head * R + rr) * n + lane];
  float2 o[kMergeFew];
#pragma unroll
  for (int s = 0; s < kMergeFew; ++s) {
    o[s] = make_float2(0.f, 0.f);
    if (s < n) o[s] = base[(size_t)s * sstride];
  }
  const float w = split_weight(ml.x, wave_max(ml.x)), den = wave_sum(w * ml.y);
  float2 num[kMergeParts];
#pragma unroll
  for (int p = 0; p < kMergeParts; ++p) num[p] = make_float2(0.f, 0.f);
#pragma unroll
  for (int s = 0; s < kMergeFew; ++s) {
    if (s < n) {
      const float ws = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(w), s));
      num[s % kMergeParts].x += ws * o[s].x;
      num[s % kMergeParts].y += ws * o[s].y;
    }
  }
#pragma unroll
  for (int p = 1; p < kMergeParts; ++p) {
    num[0].x += num[p].x;
    num[0].y += num[p].y;
  }
  const int c = rr / a.grp, gi = rr - c * a.grp;
  uint16_t* out = a.O + ((size_t)c * a.n_q_heads + head * a.grp + gi) * 128 + part_channel(2 * lane);
  out[0] = f32_to_bf16(num[0].x / den);
  out[1] = f32_to_bf16(num[0].y / den);
}

template <class BATCH>
static int launch_merge(cas_ctx* ctx, const BATCH& b, int max_r, int max_split, int n) {
  const int heads = attn_common(b).g.n_kv_heads;
  if (max_split <= kMergeFew)
    hipLaunchKernelGGL(attn_merge_few_kernel<BATCH>, dim3((max_r + 3) / 4, heads, n), dim3(256), 0, ctx->stream, b);
  else
    hipLaunchKernelGGL(attn_merge_kernel<BATCH>, dim3(max_r, heads, 2 * n), dim3(512), 0, ctx->stream, b);
  CAS_HIP(ctx, hipGetLastError());
  return CAS_OK;
}

static void set_group(AttnArgs& a, int grp) {
  a.grp = grp;
  a.grp_inv = grp > 0 ? (65536u + (uint32_t)grp - 1u) / (uint32_t)grp : 0u;
}

static int launch_partial(cas_ctx* ctx, const AttnBatch& b, int MT, int full, dim3 grid) {
  if (b.common.g.mx) {
    if (full)
      return MT == 1   ? launch_mt<1, true, true>(ctx, b, grid)
             : MT == 2 ? launch_mt<2, true, true>(ctx, b, grid)
             : MT == 3 ? launch_mt<3, true, true>(ctx, b, grid)
             : MT == 4 ? launch_mt<4, true, true>(ctx, b, grid)
                       : launch_mt<5, true, true>(ctx, b, grid);
    return MT == 1   ? launch_mt<1, false, true>(ctx, b, grid)
           : MT == 2 ? launch_mt<2, false, true>(ctx, b, grid)
                     : launch_mt<3, false, true>(ctx, b, grid);
  }
  if (full)
    return MT == 1   ? launch_mt<1, true>(ctx, b, grid)
           : MT == 2 ? launch_mt<2, true>(ctx, b, grid)
           : MT == 3 ? launch_mt<3, true>(ctx, b, grid)
           : MT == 4 ? launch_mt<4, true>(ctx, b, grid)
                     : launch_mt<5, true>(ctx, b, grid);
  return MT == 1   ? launch_mt<1, false>(ctx, b, grid)
         : MT == 2 ? launch_mt<2, false>(ctx, b, grid)
                   : launch_mt<3, false>(ctx, b, grid);
}

static void set_common(AttnArgs& a, const cas_kv* kv, const AttnCall& c) {
  a.g = kv->geom;
  a.spec_pool = (const uint32_t*)kv->d_spec;
  a.verif_pool = (const uint32_t*)kv->d_verif;
  a.layer = c.layer;
  a.n_q_heads = c.n_q_heads;
  set_group(a, c.n_q_heads / kv->geom.n_kv_heads);
  a.ystride = c.ystride; a.rope = c.rope;
  a.scale = 0.08838834764831845f;  // 1 / sqrt(128)
  a.pages_per_split = kPagesPerSplit;  // fixed: a query's value must not depend on the length
}

// bytes of committed positions (bitmap + spec (+ lo + pruned) of K and V) and of plain bf16 in-flight ones
static double attn_bytes(const KvGeom& g, int full, double len, double n_new) {
  return 2.0 * g.n_kv_heads * (4.0 * (4 + g.mx + g.sw + (full ? g.lw + g.pw : 0)) * len + 256.0 * n_new);
}

// Up to kAttnBatch sequences of one pass in one pair of launches (same layer, same form, same
// number of query heads); every sequence gets exactly what a launch of its own would give it.
// ws / ws_bytes: device memory for the per-split partial results; prof: bracket the launch with
// events when the context's measurement hooks are on (creates events: not for callers that may
// not allocate).
static int launch_attention_group(cas_ctx* ctx, cas_kv* kv, const AttnCall* calls, int n, void* ws, size_t ws_bytes,
                                  size_t* ws_used, bool prof) {
  const KvGeom& g = kv->geom;
  const AttnCall& c0 = calls[0];
  AttnBatch b{};
  AttnArgs& a = b.common;
  set_common(a, kv, c0);
  int max_r = 0, max_split = 0;
  double bytes = 0.0;
  for (int i = 0; i < n; ++i) {
    const AttnCall& c = calls[i];
    if (c.layer != c0.layer || c.full != c0.full || c.n_q_heads != c0.n_q_heads || c.ystride != c0.ystride ||
        c.rope != c0.rope || (c.qkv == nullptr) != (c0.qkv == nullptr))
      return CAS_EINVAL;
    AttnSeq& q = b.s[i];
    q.page_row = kv->d_page_table + (size_t)c.seq * g.max_pages_per_seq;
    q.len = c.len >= 0 ? c.len : kv->h_len[c.seq];
    q.Q = c.Q; q.ncols = c.ncols;
    q.Knew = c.Knew; q.Vnew = c.Vnew; q.n_new = c.n_new;
    q.qkv = c.qkv; q.slot0 = c.slot0;
    q.Kslot = c.Kslot; q.Vslot = c.Vslot;
    q.O = c.O;
    const int R = c.ncols * a.grp;
    const int MT = (R + 15) / 16;
    if (MT < 1 || MT > (c.full ? 5 : 3) || c.n_new > kPT || c.n_new < c.ncols || c.ncols > kMaxCols) return CAS_EINVAL;
    const int pages = (q.len + q.n_new + kPT - 1) / kPT;
    if (pages > g.max_pages_per_seq) return CAS_ENOMEM;
    q.nsplit = (pages + kPagesPerSplit - 1) / kPagesPerSplit;
    const size_t need = sizeof(float) * (size_t)q.nsplit * g.n_kv_heads * R * kPartStride;
    if (!ws || *ws_used + need > ws_bytes) return CAS_ENOMEM;
    q.part = (float*)((char*)ws + *ws_used);
    *ws_used += (need + 255) / 256 * 256;
    max_r = std::max(max_r, R);
    max_split = std::max(max_split, q.nsplit);
    bytes += attn_bytes(g, c.full, q.len, q.n_new);
  }
  const int MT = (max_r + 15) / 16;
  int rc;
  {
    ProfScope scope(prof ? ctx : nullptr, c0.full ? PROF_ATTN_VERIFY : PROF_ATTN_DRAFT, bytes);
    rc = launch_partial(ctx, b, MT, c0.full, dim3(max_split, g.n_kv_heads, n));
  }
  if (rc != CAS_OK) return rc;
  return launch_merge(ctx, b, max_r, max_split, n);
}

int launch_attention_batch(cas_ctx* ctx, cas_kv* kv, const AttnCall* calls, int n) {
  if (n < 1) return CAS_OK;
  // the launches of a group follow those of the group before on the stream, so every group
  // starts at the beginning of the workspace again
  for (int i = 0; i < n; i += kAttnBatch) {
    size_t ws_used = 0;
    const int rc = launch_attention_group(ctx, kv, calls + i, std::min(kAttnBatch, n - i), ctx->d_ws, ctx->ws_bytes,
                                          &ws_used, true);
    if (rc != CAS_OK) return rc;
  }
  return CAS_OK;
}

// By the query rows of a run, as for a call of its own: a small group with shared exponents, or a workspace too small for
// longer runs, has 16 rows in runs of 16 columns, and over 8000 positions of 32 kv heads products for 64 rows make the
// attention of a prompt take 1.3 times as long (shared exponents) and 1.37 times (raw) as the calls do.
static int launch_runs(cas_ctx* ctx, const AttnRuns& b, int MT, dim3 grid) {
  if (b.first.g.mx)
    return MT == 1   ? launch_mt<1, true, true>(ctx, b, grid)
           : MT == 2 ? launch_mt<2, true, true>(ctx, b, grid)
           : MT == 3 ? launch_mt<3, true, true>(ctx, b, grid)
           : MT == 4 ? launch_mt<4, true, true>(ctx, b, grid)
                     : launch_mt<5, true, true>(ctx, b, grid);
  return MT == 1   ? launch_mt<1, true, false>(ctx, b, grid)
         : MT == 2 ? launch_mt<2, true, false>(ctx, b, grid)
         : MT == 3 ? launch_mt<3, true, false>(ctx, b, grid)
                   : launch_mt<4, true, false>(ctx, b, grid);
}

// A call of c.ncols columns in runs of `run` columns, each as a call of its own whose c.len grows by the columns
// before it.  One run of 16 columns leaves most of the chip idle (up to 8 pages x 8 heads for a prompt's first 512
// positions), so as many run together as the workspace holds the partial results of: for 508 columns of the 8B shape
// 38 + 11 us per layer (both kernels) in one launch of 32 runs, 8 x (16 + 11) in launches of four.
int launch_attention_runs(cas_ctx* ctx, cas_kv* kv, const AttnCall& c, int run, void* ws, size_t ws_bytes) {
  const KvGeom& g = kv->geom;
  AttnRuns b{};
  AttnArgs& a = b.first;
  set_common(a, kv, c);
  a.page_row = kv->d_page_table + (size_t)c.seq * g.max_pages_per_seq;
  run = std::min(run, c.ncols);
  const int max_r = run * a.grp;
  if (run < 1 || run > kPT || !c.full || c.qkv || max_r > (g.mx ? 80 : 64) || c.len < 0) return CAS_EINVAL;
  if ((c.len + c.ncols + kPT - 1) / kPT > g.max_pages_per_seq) return CAS_ENOMEM;
  const size_t page_bytes = sizeof(float) * (size_t)c.n_q_heads * run * kPartStride;
  b.run_cols = run;
  a.part = (float*)ws;
  for (int c0 = 0; c0 < c.ncols;) {
    size_t pages = 0;
    int n = 0, end = c0, split = 0;
    double bytes = 0.0;
    for (; n < kAttnRuns && end < c.ncols; ++n) {
      const int cols = std::min(run, c.ncols - end), p = (c.len + end + cols + kPT - 1) / kPT;
      if ((pages + p) * page_bytes > ws_bytes) break;
      bytes += attn_bytes(g, 1, c.len + end, cols);
      b.run_page[n] = (uint32_t)pages;
      pages += p;
      end += cols;
      split = p;
    }
    if (n == 0) return CAS_ENOMEM;
    b.cols = end - c0;
    a.len = c.len + c0;
    a.Q = c.Q + (size_t)c0 * c.n_q_heads * 128; a.O = c.O + (size_t)c0 * c.n_q_heads * 128;
    a.Knew = c.Knew + (size_t)c0 * g.n_kv_heads * 128; a.Vnew = c.Vnew + (size_t)c0 * g.n_kv_heads * 128;
    const dim3 grid(split, g.n_kv_heads, n);
    int rc;
    {
      ProfScope scope(ctx, PROF_ATTN_VERIFY, bytes);
      rc = launch_runs(ctx, b, (max_r + 15) / 16, grid);
    }
    if (rc == CAS_OK) rc = launch_merge(ctx, b, max_r, split, n);
    if (rc != CAS_OK) return rc;
    c0 = end;
  }
  return CAS_OK;
}

int launch_attention(cas_ctx* ctx, cas_kv* kv, const AttnCall& c) { return launch_attention_batch(ctx, kv, &c, 1); }

// Plain bf16 attention of one decode step over an UNCOMPRESSED cache (the BFloat16 baseline, for
// context figures): the same kernels with no committed position in any pool; the cache rows play
// the part of the in-flight vectors, which the kernels take as plain bf16.  Kc, Vc:
// [max_pos][n_kv_heads][128], positions 0 .. len-1 filled; the k, v of the new token (position
// len) are split from the fp32 projection `qkv`, rotated and stored at row len.
int launch_attention_dense(cas_ctx* ctx, int n_kv_heads, int n_q_heads, uint16_t* Kc, uint16_t* Vc, int len,
                           const float* qkv, int ystride, const float* rope, uint16_t* O) {
  if (n_kv_heads < 1 || n_q_heads % n_kv_heads != 0 || len < 0 || !Kc || !Vc || !qkv || !rope || !O) return CAS_EINVAL;
  AttnBatch b{};
  AttnArgs& a = b.common;
  a.g = KvGeom{};
  a.g.n_kv_heads = n_kv_heads; a.g.page_tokens = kPT; a.g.n_pages = 1;
  a.layer = 0;
  a.n_q_heads = n_q_heads;
  set_group(a, n_q_heads / n_kv_heads);
  a.ystride = ystride; a.rope = rope;
  a.scale = 0.08838834764831845f;
  a.pages_per_split = kPagesPerSplit;
  if (a.grp > 16) return CAS_ENOTSUP;
  AttnSeq& q = b.s[0];
  q.page_row = nullptr;  // never consulted: no position is committed to a pool
  q.len = 0; q.ncols = 1; q.n_new = len + 1; q.slot0 = len;
  q.Knew = Kc; q.Vnew = Vc; q.Kslot = Kc; q.Vslot = Vc;
  q.qkv = qkv; q.Q = nullptr; q.O = O;
  q.nsplit = (len + 1 + kPT - 1) / kPT;
  const size_t need = sizeof(float) * (size_t)q.nsplit * n_kv_heads * a.grp * kPartStride;
  if (!ctx->d_ws || need > ctx->ws_bytes) return CAS_ENOMEM;
  q.part = (float*)ctx->d_ws;
  const int rc = launch_mt<1, false>(ctx, b, dim3(q.nsplit, n_kv_heads, 1));
  if (rc != CAS_OK) return rc;
  return launch_merge(ctx, b, a.grp, q.nsplit, 1);
}

// ---- the variant for callers that cannot allocate: the partial results live in a fixed array of
// the library's own instead of a workspace the caller had to obtain.  Every GPU holds its own copy
// of the array at its own address; the address is looked up once per device, with that device
// current, and only that pointer (never the array's name) is handed to kernels.
constexpr size_t kAttnScratchBytes = 32u << 20;
static __device__ __align__(256) unsigned char scratch[kAttnScratchBytes];
constexpr int kMaxDevices = 64;
static std::atomic<void*> g_scratch_ptr[kMaxDevices];

size_t attention_static_capacity() { return kAttnScratchBytes; }

int launch_attention_static(cas_ctx* ctx, cas_kv* kv, const AttnCall& c) {
  int dev = -1;
  CAS_HIP(ctx, hipGetDevice(&dev));
  if (dev != ctx->device || dev < 0 || dev >= kMaxDevices) return CAS_EINVAL;  // the context's device must be current
  void* ptr = g_scratch_ptr[dev].load(std::memory_order_acquire);
  if (!ptr) {
    CAS_HIP(ctx, hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
    if (!ptr) return CAS_EHIP;
    g_scratch_ptr[dev].store(ptr, std::memory_order_release);  // two threads racing store the same address
  }
  size_t ws_used = 0;
  // nothing in the array has to start at zero: every split writes its whole record before the
  // merge kernel, which follows on the same stream, reads exactly the records of this call
  return launch_attention_group(ctx, kv, &c, 1, ptr, kAttnScratchBytes, &ws_used, false);
}

}  // namespace cas
