// Weight formatting (selection + truncation + split + pack) and dense reconstruction.
//
// Encode follows Sec. 4.2 of the paper: per output row the K best scores |W_ij| * a_j are the
// speculation group, their low t mantissa bits and all other values are the verification
// group (Sec. 4.1).  Equal scores are granted in ascending column order.
#include "cas_device.hpp"
#include "cas_internal.hpp"

namespace cas {

struct CodecArgs {
  int64_t rows, cols, ld;
  int K, t, bw, sw, lw, pw;
  uint32_t* bitmap;
  uint32_t* spec;
  uint32_t* lo;
  uint32_t* pruned;
};

// The comparison key of one value: its score as an unsigned pattern (a NaN score ranks above every finite one).
__device__ __forceinline__ uint32_t score_of(uint32_t w, bool weighted, float act) {
  const uint32_t mag = w & 0x7FFFu;
  if (!weighted) return mag;
  const float s = __fmul_rn(__uint_as_float(mag << 16), act);
  return (s != s) ? 0x7FFFFFFFu : __float_as_uint(s);
}

// One workgroup of NW = blockDim / 64 waves formats one row; a lane owns P pieces of 8
// consecutive columns, piece (q, wave, lane) being columns 8 ((q NW + wave) 64 + lane) ..+7, so the row and
// the norms come in with 16-byte loads and are read from memory once: values and keys stay in registers (with 10
// pieces, rows of more than 65536 columns, 98 of the 128 registers that sixteen waves leave a lane spill).
//
//   1. The K-th largest key is found bit by bit: a wave counts the keys >= a candidate with ballots (one
//      compare per key, the counting runs on the scalar unit), the waves of a row add their counts in LDS.
//      The search ends early when exactly K keys are left above the candidate.
//   2. Prefix sums over (piece, wave, lane), which is column order, rank the kept values; equal keys at the
//      threshold are granted in column order.  A value is written once, as 16 bits, to its place in the
//      row's kept or pruned list in LDS.
//   3. A thread packs 32 consecutive kept values into the FW words of the spec stream and the T words of the
//      lo stream that they fill exactly; the pruned list already is the pruned stream.
//
// Bound by the issue of vector instructions, the compares of step 1 (about 22 of them per value) above all:
// counters of 28672 x 4096 with norms have them in 71 % of the cycles that the CUs are busy (92 % of the launch);
// scalar instructions, one a cycle for the four SIMDs, in 61 %.  269 us, 1.8 TB/s of input and output; radix
// selection through histograms in LDS, whose atomics met in the few exponents that a row holds, took 2602 us.
template <int T, int P>
__global__ __launch_bounds__(1024) void encode_rows_kernel(const uint16_t* __restrict__ W,
                                                           const float* __restrict__ act, CodecArgs a) {
  constexpr int FW = 16 - T;
  extern __shared__ uint16_t vals[];  // [kpad] kept values of the row, then the pruned ones
  __shared__ int wave_cnt[2][16];
  __shared__ uint32_t tot_gt[P * 16], tot_eq[P * 16];

  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nthr = blockDim.x, NW = nthr >> 6;
  const int cols = (int)a.cols, K = a.K, kpad = (K + 31) & ~31, npruned = cols - K;
  const bool weighted = act != nullptr;
  if (blockIdx.x == 0 && tid < 64) {  // the slack kernels may over-read must hold finite values
    a.spec[a.rows * a.sw + tid] = 0;
    a.lo[a.rows * a.lw + tid] = 0;
    a.pruned[a.rows * a.pw + tid] = 0;
  }
  const int64_t row = blockIdx.x;
  const uint16_t* wr = W + row * a.ld;
  uint32_t raw[P][4], key[P][8];
#pragma unroll
  for (int q = 0; q < P; ++q) {
    const int col = ((q * NW + wv) * 64 + lane) * 8;
#pragma unroll
    for (int e = 0; e < 8; ++e) key[q][e] = 0u;
#pragma unroll
    for (int e = 0; e < 4; ++e) raw[q][e] = 0u;
    if (col + 8 <= cols) {  // a row may start at any multiple of 2 bytes
      __builtin_memcpy(raw[q], wr + col, 16);
      if (weighted) __builtin_memcpy(key[q], act + col, 32);
    } else if (col < cols) {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        if (col + e < cols) {
          raw[q][e >> 1] |= (uint32_t)wr[col + e] << (16 * (e & 1));
          if (weighted) key[q][e] = __float_as_uint(act[col + e]);
        }
      }
    }
  }
#pragma unroll
  for (int q = 0; q < P; ++q) {
    // columns past the end have value 0 and norm 0, hence the smallest key: no candidate counts them
#pragma unroll
    for (int e = 0; e < 8; ++e)
      key[q][e] = score_of(raw[q][e >> 1] >> (16 * (e & 1)), weighted, __uint_as_float(key[q][e]));
    __builtin_amdgcn_sched_barrier(0);
  }
  // ---- 1. thr: the largest value that at least K keys reach
  int buf = 0;
  auto count_ge = [&](uint32_t cand) -> int {
    int c = 0;
#pragma unroll
    for (int q = 0; q < P; ++q) {
#pragma unroll
      for (int e = 0; e < 8; ++e) c += __popcll(__builtin_amdgcn_ballot_w64(key[q][e] >= cand));
      __builtin_amdgcn_sched_barrier(0);  // eight masks at a time: all of them together do not fit the scalar registers
    }
    if (NW > 1) {  // two sets of slots: one barrier per count keeps a fast wave out of the set being read
      if (lane == 0) wave_cnt[buf][wv] = c;
      __syncthreads();
      c = 0;
      for (int w = 0; w < NW; ++w) c += wave_cnt[buf][w];
      c = __builtin_amdgcn_readfirstlane(c);
      buf ^= 1;
    }
    return c;
  };
  uint32_t thr = 0;
  bool exact = K == cols;  // exactly K keys are >= thr
  int need = 0;            // how many of the keys equal to thr are kept, when not exact
  if (K == 0) {
    thr = 0xFFFFFFFFu;     // no key is that large: the largest are those of -Inf norms, 0xFF800000
    exact = true;
  } else if (!exact) {
    for (int bit = weighted ? 31 : 14; bit >= 0 && !exact; --bit) {
      const uint32_t cand = thr | (1u << bit);
      const int c = count_ge(cand);
      if (c >= K) {
        thr = cand;
        exact = c == K;
      }
    }
    if (!exact) need = K - count_ge(thr + 1u);
  }
  // ---- 2. ranks
  const uint32_t sure = exact ? thr : thr + 1u, tied = thr;
  uint32_t gt[P], excl[P];  // bit e: kept for certain, bit 8 + e: equal to thr; counts before the lane's piece
#pragma unroll
  for (int q = 0; q < P; ++q) {
    const int col = ((q * NW + wv) * 64 + lane) * 8;
    uint32_t g = 0, eq = 0;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      g |= (uint32_t)(key[q][e] >= sure) << e;
      eq |= (uint32_t)(key[q][e] == tied) << e;
    }
    const uint32_t in = cols - col >= 8 ? 0xFFu : (cols > col ? (1u << (cols - col)) - 1u : 0u);
    g &= in;
    eq &= exact ? 0u : in;
    gt[q] = g | (eq << 8);
    __builtin_amdgcn_sched_barrier(0);
    const int c = __popc(g) | (__popc(eq) << 16);
    const int incl = wave_incl_scan(c);
    excl[q] = (uint32_t)(incl - c);
    const uint32_t total = (uint32_t)__builtin_amdgcn_readlane(incl, 63);
    if (lane == 0) {
      tot_gt[q * NW + wv] = total & 0xFFFFu;
      tot_eq[q * NW + wv] = total >> 16;
    }
  }
  __syncthreads();
  uint32_t base_gt = 0, base_eq = 0;
  int next = 0;  // entries of the totals already added to the bases
#pragma unroll
  for (int q = 0; q < P; ++q) {
    for (; next < q * NW + wv; ++next) {
      base_gt += tot_gt[next];
      base_eq += tot_eq[next];
    }
    const int piece = (q * NW + wv) * 64 + lane, col = piece * 8;
    uint32_t eq_run = base_eq + (excl[q] >> 16);
    uint32_t p = base_gt + (excl[q] & 0xFFFFu) + min(eq_run, (uint32_t)need);  // kept values before the piece
    uint32_t m = 0;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      bool kept = (gt[q] >> e) & 1u;
      if ((gt[q] >> (8 + e)) & 1u) {
        kept = eq_run < (uint32_t)need;
        ++eq_run;
      }
      // columns past the end go to a slot that nothing reads
      const uint32_t at = kept ? p : min((uint32_t)(kpad + col + e) - p, (uint32_t)(kpad + npruned + 1));
      vals[at] = (uint16_t)(raw[q][e >> 1] >> (16 * (e & 1)));
      m |= (uint32_t)kept << e;
      p += kept ? 1u : 0u;
    }
    __builtin_amdgcn_sched_barrier(0);
    if (piece < 4 * a.bw) reinterpret_cast<uint8_t*>(a.bitmap + row * a.bw)[piece] = (uint8_t)m;
  }
  if (tid < kpad - K) vals[K + tid] = 0;
  if (tid == 0 && (npruned & 1)) vals[kpad + npruned] = 0;
  __syncthreads();
  // ---- 3. streams
  for (int g = tid; g < (kpad >> 5); g += nthr) {
    uint32_t v[16], sp[FW], lo[T > 0 ? T : 1];
    __builtin_memcpy(v, __builtin_assume_aligned(vals + 32 * g, 16), 64);
#pragma unroll
    for (int i = 0; i < FW; ++i) sp[i] = 0;
#pragma unroll
    for (int i = 0; i < (T > 0 ? T : 1); ++i) lo[i] = 0;
    static_for<0, 32>([&](auto I) {
      constexpr int i = decltype(I)::value, bit = i * FW, w = bit >> 5, sh = bit & 31;
      const uint32_t x = (v[i >> 1] >> (16 * (i & 1))) & 0xFFFFu, hi = x >> T;
      sp[w] |= hi << sh;
      if constexpr (sh + FW > 32) sp[w + 1] |= hi >> (32 - sh);
      if constexpr (T > 0) {
        constexpr int lb = i * T, lwd = lb >> 5, lsh = lb & 31;
        const uint32_t l = x & ((1u << T) - 1u);
        lo[lwd] |= l << lsh;
        if constexpr (lsh + T > 32) lo[lwd + 1] |= l >> (32 - lsh);
      }
    });
    uint32_t* ds = a.spec + row * a.sw + g * FW;
    if ((g + 1) * FW <= a.sw) {
      __builtin_memcpy(ds, sp, 4 * FW);
    } else {
#pragma unroll
      for (int i = 0; i < FW; ++i)
        if (g * FW + i < a.sw) ds[i] = sp[i];
    }
    if constexpr (T > 0) {
      uint32_t* dl = a.lo + row * a.lw + g * T;
      if ((g + 1) * T <= a.lw) {
        __builtin_memcpy(dl, lo, 4 * T);
      } else {
#pragma unroll
        for (int i = 0; i < T; ++i)
          if (g * T + i < a.lw) dl[i] = lo[i];
      }
    }
  }
  const uint32_t* pl = reinterpret_cast<const uint32_t*>(vals + kpad);
  for (int i = tid; i < a.pw; i += nthr) a.pruned[row * a.pw + i] = pl[i];
}

// Dense reconstruction of one row per workgroup; full == 0 gives the zero-padded draft view.
__global__ __launch_bounds__(256) void decode_rows_kernel(CodecArgs a, uint16_t* __restrict__ out, int full) {
  extern __shared__ uint32_t smem[];
  uint32_t* pre = smem;  // bw
  const int tid = threadIdx.x;
  const int cols = (int)a.cols;
  const int fw = 16 - a.t;
  for (int64_t row = blockIdx.x; row < a.rows; row += gridDim.x) {
    const uint32_t* bm = a.bitmap + row * a.bw;
    for (int wd = tid; wd < a.bw; wd += 256) pre[wd] = __popc(bm[wd]);
    __syncthreads();
    if (tid == 0) {
      uint32_t s = 0;
      for (int wd = 0; wd < a.bw; ++wd) {
        uint32_t t = pre[wd];
        pre[wd] = s;
        s += t;
      }
    }
    __syncthreads();
    const uint32_t* sp = a.spec + row * a.sw;
    const uint32_t* lo = a.lo + row * a.lw;
    const uint32_t* pr = a.pruned + row * a.pw;
    for (int wd = tid; wd < a.bw; wd += 256) {
      uint32_t m = bm[wd];
      uint32_t p = pre[wd], u = (uint32_t)wd * 32u - p;
      for (int c = 0; c < 32; ++c) {
        int j = wd * 32 + c;
        if (j >= cols) break;
        uint32_t v;
        if ((m >> c) & 1u) {
          v = read_field(sp, p * fw, fw) << a.t;
          if (full && a.t) v |= read_field(lo, p * a.t, a.t);
          ++p;
        } else {
          v = full ? read_field(pr, u * 16, 16) : 0u;
          ++u;
        }
        out[row * a.ld + j] = (uint16_t)v;
      }
    }
    __syncthreads();
  }
}

static CodecArgs make_args(const cas_wdesc& d, const void* spec, const void* verif, int64_t ld) {
  CodecArgs a;
  a.rows = d.rows; a.cols = d.cols; a.ld = ld;
  a.K = d.K; a.t = d.t; a.bw = d.bw; a.sw = d.sw; a.lw = d.lw; a.pw = d.pw;
  char* s = (char*)spec;
  char* v = (char*)verif;
  a.bitmap = (uint32_t*)(s + d.off_bitmap);
  a.spec = (uint32_t*)(s + d.off_spec);
  a.lo = v ? (uint32_t*)(v + d.off_lo) : nullptr;
  a.pruned = v ? (uint32_t*)(v + d.off_pruned) : nullptr;
  return a;
}

// One launch takes the rows whose threads number less than 2^32, the limit of a grid; a matrix of more rows (2^26
// of up to 4096 columns) takes several.
template <int T, int P>
static int launch_encode_instance(cas_ctx* ctx, const uint16_t* W, const float* act, CodecArgs a, int waves) {
  const size_t lds = sizeof(uint16_t) * ((size_t)((a.K + 31) & ~31) + (size_t)(a.cols - a.K) + 2);
  static LdsLimit lim;
  const int rc = allow_lds(ctx, (const void*)encode_rows_kernel<T, P>, lds, lim);
  if (rc != CAS_OK) return rc;
  const int64_t most = 0xFFFFFFFFll / (64 * waves);
  while (a.rows > 0) {
    const int64_t n = std::min(a.rows, most);
    hipLaunchKernelGGL((encode_rows_kernel<T, P>), dim3((unsigned)n), dim3(64 * waves), lds, ctx->stream, W, act, a);
    CAS_HIP(ctx, hipGetLastError());
    a.rows -= n;  // the slack behind the streams stays where it is
    W += n * a.ld;
    a.bitmap += n * a.bw;
    a.spec += n * a.sw;
    a.lo += n * a.lw;
    a.pruned += n * a.pw;
  }
  return CAS_OK;
}

// 512 columns per wave and piece.  One wave of 2, 4 or 8 pieces takes rows of up to 4096 columns (no
// barriers in the search); longer rows go to as many waves of 8 pieces as they need, and those beyond 16 of
// them (65536 columns) to 16 waves of 10 pieces, which hold 81920: more than launch_encode_weight lets through.
template <int T>
static int launch_encode_t(cas_ctx* ctx, const uint16_t* W, const float* act, const CodecArgs& a) {
  if (a.cols <= 1024) return launch_encode_instance<T, 2>(ctx, W, act, a, 1);
  if (a.cols <= 2048) return launch_encode_instance<T, 4>(ctx, W, act, a, 1);
  if (a.cols <= 65536) return launch_encode_instance<T, 8>(ctx, W, act, a, (int)((a.cols + 4095) / 4096));
  return launch_encode_instance<T, 10>(ctx, W, act, a, 16);
}

int launch_encode_weight(cas_ctx* ctx, const uint16_t* W, int64_t ld, const float* act, const cas_wdesc& d,
                         void* spec, void* verif) {
  CodecArgs a = make_args(d, spec, verif, ld);
  // The longest row that is taken: its streams, two counters per bitmap word and 1 KB within the LDS of a
  // workgroup, 72366 columns at most.  The kernel itself needs two bytes per column and a little.
  if (sizeof(uint32_t) * ((size_t)d.sw + d.lw + d.pw + 256 + 2 * (size_t)d.bw) > (size_t)ctx->lds_max) return CAS_ENOTSUP;
  if (d.rows < 1) return CAS_OK;
  switch (d.t) {
    case 0: return launch_encode_t<0>(ctx, W, act, a);
    case 1: return launch_encode_t<1>(ctx, W, act, a);
    case 2: return launch_encode_t<2>(ctx, W, act, a);
    case 3: return launch_encode_t<3>(ctx, W, act, a);
    case 4: return launch_encode_t<4>(ctx, W, act, a);
    case 5: return launch_encode_t<5>(ctx, W, act, a);
    case 6: return launch_encode_t<6>(ctx, W, act, a);
    case 7: return launch_encode_t<7>(ctx, W, act, a);
    default: return CAS_EINVAL;
  }
}

int launch_decode_weight(cas_ctx* ctx, const cas_wdesc& d, const void* spec, const void* verif, uint16_t* out,
                         int64_t ld) {
  CodecArgs a = make_args(d, spec, verif, ld);
  size_t lds = sizeof(uint32_t) * (size_t)d.bw;
  int grid = (int)std::min<int64_t>(d.rows, (int64_t)ctx->num_cu * 8);
  if (grid < 1) return CAS_OK;
  hipLaunchKernelGGL(decode_rows_kernel, dim3(grid), dim3(256), lds, ctx->stream, a, out, verif ? 1 : 0);
  CAS_HIP(ctx, hipGetLastError());
  return CAS_OK;
}

}  // namespace cas
