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

// One workgroup of NW = blockDim / 64 waves formats one row; a lane owns P pieces of 8
// consecutive columns, piece (q, wave, lane) being columns 8 ((q NW + wave) 64 + lane) ..+7, so the row and
// the norms come in with 16-byte loads and are read from memory once: values and keys stay in registers (with 10
// pieces, rows of more than 65536 columns, 79 of the 128 registers that sixteen waves leave a lane spill).
//
//   1. The threshold is a value that exactly K keys reach, or the K-th largest key itself.  A lane counts its own keys,
//      two instructions a key; the sum goes over the lanes, and in LDS over the waves of the row.  Long rows, and
//      matrices of many rows with norms: it lies between two values whose counts are known; a sample of 64 keys gives
//      the first of them, and from there on the next candidate is where a straight line between the two counts meets
//      K.  Seven counts find it among 4096 keys, where a search bit by bit takes 19 (with norms; five instead of 16
//      without).  The others bit by bit (search_bits).
//   2. Where keys equal the threshold, the first in column order of them are raised above it.  Prefix sums over
//      (piece, wave, lane), which is column order, rank the kept values.  A value is written once, as 16 bits, to its place in the
//      row's kept or pruned list in LDS.
//   3. A thread packs 32 consecutive kept values into the FW words of the spec stream and the T words of the
//      lo stream that they fill exactly; the pruned list already is the pruned stream.
//
// Bound by the issue of instructions, some 45 per value, and by the start of a row, when its wave waits for its
// loads: all of them are in flight together (a branch around each had them wait one by one, 46 us of the launch).
// 28672 x 4096 with norms, which is more than the caches hold, 160 us, 3.0 TB/s of input and output (283 with the search
// bit by bit and branched loads), without 158 (234); 8192 x 14336, four waves a row, 199 (381).  Radix selection
// through histograms in LDS, whose atomics met in the few exponents that a row holds, took 2602 us; counting
// with ballots, which are three instructions a key, 231 where this took 170.
constexpr int kSampleStep = 4;       // places of the sample on either side of the expected one: one standard deviation
constexpr int kInterpolations = 12;  // counts after which the rest of the interval is halved
constexpr unsigned kFewRows = 4096;  // four waves of one row each for every SIMD

// Whether a row's threshold is found bit by bit.  Such a count has next to nothing to work out before it, and there are
// at most 17 of them (34 with norms) whatever the values are; the line needs fewer on average, but some rows need as many
// and each takes longer.  Bit by bit / by the line, us.  Rows of up to 1024 columns without norms: 512 x 256 7.8 / 8.7,
// 28672 x 1000 61.2 / 56.4; values that are whole numbers up to 10, so that most keys are equal: 7.9 / 11.6 and
// 64.1 / 70.2.  With norms, where such rows lack a full sample or a wave has its SIMD to itself or nearly so: 512 x 256
// 9.1 / 10.9, 8192 x 256 21.8 / 21.8, 2048 x 1000 11.1 / 11.5 (25 % kept: 11.7 / 13.3), 4096 x 512 15.5 / 15.5 (14.8 / 16.1),
// 8192 x 768 23.8 / 22.9, 28672 x 1000 66.3 / 58.7.  Longer rows: 256 x 2000 without norms 12.9 / 10.4, where it is only
// such whole numbers 12.9 / 14.9; 4096 x 4096 43.2 / 32.7 and 43.2 / 42.4.
template <int P>
__device__ __forceinline__ bool search_bits(bool weighted, int cols) {
  return P == 2 && (!weighted || cols < 512 || gridDim.x <= kFewRows);
}

template <int T, int P>
__global__ __launch_bounds__(1024) void encode_rows_kernel(const uint16_t* __restrict__ W,
                                                           const float* __restrict__ act, CodecArgs a) {
  constexpr int FW = 16 - T;
  extern __shared__ uint16_t vals[];  // [kpad] kept values of the row, then the pruned ones
  __shared__ int wave_cnt[2][16];
  __shared__ __attribute__((aligned(16))) uint16_t end_raw[8];
  __shared__ __attribute__((aligned(16))) float end_act[8];
  __shared__ uint32_t tot[P * 16], sample[64];

  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nthr = blockDim.x, NW = nthr >> 6;
  const int cols = (int)a.cols, K = a.K, kpad = (K + 31) & ~31, npruned = cols - K;
  const bool weighted = act != nullptr && K < cols;  // norms choose among the columns
  if (blockIdx.x == 0 && tid < 64) {  // the slack kernels may over-read must hold finite values
    a.spec[a.rows * a.sw + tid] = 0;
    a.lo[a.rows * a.lw + tid] = 0;
    a.pruned[a.rows * a.pw + tid] = 0;
  }
  const int64_t row = blockIdx.x;
  const uint16_t* wr = W + row * a.ld;
  if (cols & 7) {  // the piece that the row ends in, filled up with zeros
    const int col = (cols & ~7) + tid;
    if (tid < 8) {
      end_raw[tid] = col < cols ? wr[col] : (uint16_t)0;
      end_act[tid] = weighted && col < cols ? act[col] : 0.f;
    }
    __syncthreads();
  }
  // All loads are issued without a branch between them (a wait for each of the 3 P otherwise): lanes past the last
  // whole piece of the row read its first one and are corrected below.
  uint32_t raw[P][4], key[P][8];
  const int whole = cols & ~7;
  if (whole) {
    auto at = [&](int q) -> uint32_t {
      const int col = ((q * NW + wv) * 64 + lane) * 8;
      return col < whole ? (uint32_t)col : 0u;
    };
#pragma unroll
    for (int q = 0; q < P; ++q)  // a row may start at any multiple of 2 bytes
      __builtin_memcpy(raw[q], reinterpret_cast<const char*>(wr) + at(q) * 2u, 16);
    if (weighted) {
#pragma unroll
      for (int q = 0; q < P; ++q) __builtin_memcpy(key[q], reinterpret_cast<const char*>(act) + at(q) * 4u, 32);
    }
  }
#pragma unroll
  for (int q = 0; q < P; ++q) {
    if (((q * NW + wv) * 64 + 64) * 8 <= whole) continue;
    const int col = ((q * NW + wv) * 64 + lane) * 8;
    const bool in = col < whole, end = col == whole && whole < cols;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      uint32_t last;
      __builtin_memcpy(&last, end_raw + 2 * e, 4);
      raw[q][e] = in ? raw[q][e] : end ? last : 0u;
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) key[q][e] = in ? key[q][e] : end ? __float_as_uint(end_act[e]) : 0u;
  }
  // The comparison keys: magnitudes, or scores as unsigned patterns (a NaN score ranks above every finite one).
  // Columns past the end have value 0 and norm 0, hence the smallest key: no candidate counts them.
  if (weighted) {
#pragma unroll
    for (int q = 0; q < P; ++q) {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const uint32_t mag = e & 1 ? raw[q][e >> 1] & 0x7FFF0000u : raw[q][e >> 1] << 17 >> 1;
        const float s = __fmul_rn(__uint_as_float(mag), __uint_as_float(key[q][e]));
        const uint32_t nan = 0u - (uint32_t)(s != s);  // a select here becomes a branch per value
        key[q][e] = (nan & 0x7FFFFFFFu) | (~nan & __float_as_uint(s));
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  } else {
#pragma unroll
    for (int q = 0; q < P; ++q)
#pragma unroll
      for (int e = 0; e < 8; ++e) key[q][e] = (raw[q][e >> 1] >> (16 * (e & 1))) & 0x7FFFu;
  }
  // ---- 1. thr: a value with `need` of the keys equal to it and all the larger ones kept
  int buf = 0;
  auto count_ge = [&](uint32_t cand) -> int {
    int c = 0;
#pragma unroll
    for (int q = 0; q < P; ++q)
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        c += key[q][e] >= cand ? 1 : 0;  // two instructions; ballots took three
        asm("" : "+v"(c));               // one after the other: 64 masks at a time do not fit the scalar registers
      }
    c = __builtin_amdgcn_readlane(wave_incl_scan(c), 63);
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
  bool exact = false;  // exactly K keys are >= thr
  int need = 0;        // how many of the keys equal to thr are kept, when not exact
  if (K == 0) {
    thr = 0xFFFFFFFFu;     // no key is that large: the largest are those of -Inf norms, 0xFF800000
    exact = true;
  } else if (K == cols) {
    need = K;
  } else if (search_bits<P>(weighted, cols)) {
    int c = weighted ? count_ge(1u) : K + 1;  // with norms 32 counts would find that fewer than K keys are above 0
    if (c > K) {
      for (int bit = weighted ? 31 : 14; bit >= 0 && !exact; --bit) {
        const uint32_t cand = thr | (1u << bit);
        c = count_ge(cand);
        if (c >= K) {
          thr = cand;
          exact = c == K;
        }
      }
    }
    if (!exact) need = K - count_ge(thr + 1u);
  } else {
    // the sample: a key of every lane (of some lanes, where several waves share the row), from all its pieces
    const int per = 64 / NW;
    uint32_t mine = key[0][0];
    const int sq = NW == 1 ? lane * P >> 6 : min(lane, per - 1) * P / per;
#pragma unroll
    for (int q = 1; q < P; ++q) mine = sq == q ? key[q][0] : mine;
    if (((sq * NW + wv) * 64 + lane) * 8 >= cols || lane >= per) mine = 0xFFFFFFFFu;  // not a column of the row
    if (NW > 1) {
      if (tid < 64) sample[tid] = 0xFFFFFFFFu;
      __syncthreads();
      if (lane < per) sample[wv * per + lane] = mine;
      __syncthreads();
      mine = sample[lane];
    }
    const bool real = mine != 0xFFFFFFFFu;
    mine = real ? mine : 0u;
    const int n = __popcll(__builtin_amdgcn_ballot_w64(real));
    // ranks, largest first, of keys made different by their lane
    const uint32_t own = (weighted ? mine & ~63u : mine << 6) | (uint32_t)lane;
    int rank = 0;
#pragma unroll
    for (int j = 0; j < 64; ++j) rank += (uint32_t)__builtin_amdgcn_readlane((int)own, j) > own;
    auto ranked = [&](int i) -> uint32_t {
      const uint64_t at = __builtin_amdgcn_ballot_w64(rank == max(min(i, n - 1), 0));
      return (uint32_t)__builtin_amdgcn_readlane((int)mine, __builtin_ctzll(at));
    };
    // lo: reached by clo >= K keys; hi: by chi < K
    const uint32_t top = weighted ? 0xFFFFFFFFu : 0x8000u;
    uint32_t lo = 0, hi = top;
    int clo = cols, chi = 0;
    const int mid = (int)((float)K / (float)cols * (float)n);
    int below = kSampleStep, above = kSampleStep, last = 0;
    // Without norms few keys may hold all the values, and one end of the line would stay where it is for many counts:
    // its weight is halved with every count that the other end moves again.
    const float stay = weighted ? 1.f : 0.5f;
    float wlo = 1.f, whi = 1.f;
    for (int it = 0; hi - lo > 1u; ++it) {
      uint32_t cand;
      if (lo == 0u && mid + below < n + kSampleStep) {
        cand = ranked(mid + below);
        below *= 3;
      } else if (hi == top && mid - above > -kSampleStep) {
        cand = ranked(mid - above) + 1u;
        above *= 3;
      } else if (lo == 0u || hi == top || it >= kInterpolations) {
        cand = lo + ((hi - lo) >> 1);
      } else {
        const float dlo = (float)(clo - K) * wlo, dhi = (float)(K - chi) * whi;
        cand = lo + (uint32_t)((float)(hi - lo) * (dlo * __builtin_amdgcn_rcpf(dlo + dhi)));
      }
      cand = (uint32_t)__builtin_amdgcn_readfirstlane((int)min(max(cand, lo + 1u), hi - 1u));
      const int c = count_ge(cand);
      if (c >= K) {
        lo = cand;
        clo = c;
        exact = c == K;
        if (exact) break;
        wlo = 1.f;
        if (last > 0) whi *= stay;
        last = 1;
      } else {
        hi = cand;
        chi = c;
        whi = 1.f;
        if (last < 0) wlo *= stay;
        last = -1;
      }
    }
    thr = lo;
    need = K - chi;  // not exact: hi = lo + 1, which chi keys reach
  }
  // ---- 2. ranks
  // counts of the pieces before a wave's piece q: entries of tot that it has not added yet
  uint32_t base = 0;
  int next = 0;
  auto before = [&](int q) -> uint32_t {
    for (; next < q * NW + wv; ++next) base += tot[next];
    return base;
  };
  uint32_t rank[P];  // bits of the lane's piece, and from bit 8 on the count in front of it within the wave's
  if (!exact) {      // the first `need` of the keys equal to thr become the largest key
#pragma unroll
    for (int q = 0; q < P; ++q) {
      const int left = cols - ((q * NW + wv) * 64 + lane) * 8;
      uint32_t m = 0;
#pragma unroll
      for (int e = 0; e < 8; ++e) m |= key[q][e] == thr ? 1u << e : 0u;
      m &= left >= 8 ? 0xFFu : left > 0 ? (1u << left) - 1u : 0u;
      const int c = __popc(m), incl = wave_incl_scan(c);
      rank[q] = (uint32_t)(incl - c) << 8 | m;
      if (lane == 63) tot[q * NW + wv] = (uint32_t)incl;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < P; ++q) {
      const int grant = need - (int)(before(q) + (rank[q] >> 8));  // to the first of the piece
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const bool eq = (rank[q] >> e) & 1u;
        if (eq & ((int)__popc(rank[q] & ((1u << e) - 1u)) < grant)) key[q][e] = 0xFFFFFFFFu;
      }
    }
    __syncthreads();
    base = 0;
    next = 0;
  }
  const uint32_t sure = exact ? thr : thr + 1u;  // above 0, the key of columns past the end
#pragma unroll
  for (int q = 0; q < P; ++q) {
    uint32_t m = 0;
#pragma unroll
    for (int e = 0; e < 8; ++e) m |= key[q][e] >= sure ? 1u << e : 0u;
    const int c = __popc(m), incl = wave_incl_scan(c);
    rank[q] = (uint32_t)(incl - c) << 8 | m;
    if (lane == 63) tot[q * NW + wv] = (uint32_t)incl;
    __builtin_amdgcn_sched_barrier(0);
  }
  __syncthreads();
  uint32_t bound = (uint32_t)__builtin_amdgcn_readfirstlane((int)sure);
  asm("" : "+s"(bound));  // the comparisons are made again: 64 masks do not fit the scalar registers
#pragma unroll
  for (int q = 0; q < P; ++q) {
    const int piece = (q * NW + wv) * 64 + lane, col = piece * 8;
    uint32_t p = before(q) + (rank[q] >> 8);  // kept values before the piece
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const bool kept = key[q][e] >= bound;
      // columns past the end go to a slot that nothing reads
      const uint32_t at = kept ? p : min((uint32_t)(kpad + col + e) - p, (uint32_t)(kpad + npruned + 1));
      vals[at] = (uint16_t)(raw[q][e >> 1] >> (16 * (e & 1)));
      p += kept ? 1u : 0u;
    }
    __builtin_amdgcn_sched_barrier(0);
    if (piece < 4 * a.bw) reinterpret_cast<uint8_t*>(a.bitmap + row * a.bw)[piece] = (uint8_t)rank[q];
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
