// Kernel template of the draft GEMV, shared by the raw-exponent form (gemv_draft.hip) and the
// shared-exponent form (mx.hip); each of the two files instantiates its own set.
#pragma once
#include <algorithm>
#include "cas_device.hpp"
#include "cas_internal.hpp"

namespace cas {

struct GemvArgs {
  int rows, cols, bw, sw, nwaves;
  const uint32_t* bitmap;
  const uint32_t* spec;
  const uint16_t* x;  // [NB][cols]
  float* y;           // [NB][yld] (epilogue 0)
  int yld;            // output rows per column in y / out16 (>= rows: the launch may cover a block of rows)
  // optional fused neighbours of the linear layer
  const uint16_t* gain;  // non-null: x is first RMS-normalised with this gain (rounded to bf16)
  float eps;
  int epi;               // 0: y = W x;  1: h = bf16(h + bf16(W x));  2: act[i] = swiglu(rows 2i, 2i+1)
  uint16_t* out16;       // h [NB][yld] (epilogue 1) or act [NB][yld/2] (epilogue 2)
  // shared-exponent form only: one exponent byte per bitmap word, ew bytes per row
  const uint8_t* sexp;
  int ew;
};

template <int FW>
struct Window {
  uint32_t m;
  uint32_t sh;
  uint32_t e;  // shared exponent of the lane's word (shared-exponent form)
  uint32_t d[FW + 1];
};

struct Cursor {  // walks the (row, chunk) items of one wave in order
  int row, chunk;
  // pair == 0: rows gw, gw + nwaves, ...; pair == 1: row pairs (2u, 2u+1) for u = gw, gw + nwaves, ...
  __device__ __forceinline__ void advance(int nchunk, int nwaves, int pair) {
    if (++chunk == nchunk) {
      chunk = 0;
      row += pair ? ((row & 1) ? 2 * nwaves - 1 : 1) : nwaves;
    }
  }
};

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int kGemvThreads = 1024;  // 16 waves share one staged copy of x
constexpr int kGemvWaves = kGemvThreads / 64;

// x in LDS: fp32 where that fits; bf16 bit patterns (XH) for a batch that does not, which costs an operation per
// use and column.  The staged values are bf16-representable either way, so both give the same bits.  The kernel spends
// 73 % of its busy cycles issuing vector instructions, and two or four columns come with one (aligned) read: 28672 x 4096
// with 2 / 3 / 4 columns 37.0 / 43.6 / 40.1 us as bf16, 30.3 / 34.2 / 33.4 as fp32; 4096 x 4096 7.7 / 9.1 / 8.8 and 7.6 / 7.6 / 7.7.
// Layout: per chunk of 64 bitmap words a block [1 + 32][64 lanes][NB]; row 0 holds zeros, row
// 1 + k the values of column k of every lane's word.  A lane only ever reads entries of its own
// 4-byte column of the block, so the gathers of a wave never meet in a bank whatever positions
// the lanes are at (with one 33-entry segment per lane they collided at ~3.8 extra cycles per
// gather, which made the LDS a co-limit of the kernel).
constexpr int kXRows = 33;
template <int FW>
constexpr size_t kMagTabBytes = sizeof(float) << FW;
template <int NB>
__device__ __forceinline__ int x_index(int col) {  // index of x[col][0] in the staged layout
  const int w = col >> 5;
  return (((w >> 6) * kXRows + 1 + (col & 31)) * 64 + (w & 63)) * NB;
}
// FAR: one column of up to 4096 values, FAR chunks of 2048.  A position lies 256 bytes from the next, so it is the second
// byte of the address, and the bit search writes it there itself: one operation where the search and the address took two,
// of four cycles each (same bits).  The 8 KB of the second chunk lie behind those of the first, at an offset in the
// instruction: the two items in flight of a wave are always one of each.  A lane that has run out writes 255, a row of zeros
// that each chunk has at that distance.  What lies between is free: the sums of the norm and the table of
// magnitudes lie there, and not in static LDS: the second byte is the position only if the dynamic LDS begins at address
// 0, which the launch checks (allow_lds).  28672 x 4096 and its like are three quarters of a draft pass: a round of the 8B shape 20.02 -> 19.59
// ms, over shared exponents (8 layers) 6.30 -> 6.05 (both sides timed in turn); 4096 x 4096 at 25 %, a launch and its
// round trips for the most part, stays at 5.0 us.
constexpr int kFarZero = 64 << 10, kFarChunk = 8 << 10, kFarRed = 24 << 10, kFarTab = 32 << 10;  // bytes
// Reads of x ahead of their products.  Left to itself the compiler waits for each read before it issues the next one,
// which the waves of a full chip hide and those of a matrix of few rows do not, us, general form / FAR so / FAR with four
// ahead: 1024 x 4096 4.38 / 4.81 / 4.32, 2048 x 4096 5.1 / 5.3 / 4.9, 5120 x 2560 7.4 / 7.8 / 7.0, 6144 x 4096 8.3 / 8.6 /
// 7.9, 14336 x 4096 15.7 / 14.0 / 14.1, 28672 x 4096 27.8 / 25.8 / 24.9; over shared exponents 1024 x 4096 4.8 / 5.0 / 4.7,
// 5120 x 2560 7.6 / 8.2 / 7.5, 28672 x 4096 31.7 / 29.6 / 28.9.  Eight ahead, or groups of four or eight, are within 3 %.
constexpr int kFarAhead = 4;
__device__ __forceinline__ int far_row(int chunk, int row) { return chunk * (kFarChunk / 4) + row * 64; }  // of x
__device__ __forceinline__ int far_index(int col) { return far_row(col >> 11, col & 31) + ((col >> 5) & 63); }
// the position of the lowest set bit of m (255 if there is none) in the second byte of addr
__device__ __forceinline__ void put_lowest_bit(uint32_t& addr, uint32_t m) {
  asm("v_ffbl_b32_sdwa %0, %1 dst_sel:BYTE_1 dst_unused:UNUSED_PRESERVE src0_sel:DWORD" : "+v"(addr) : "v"(m));
}
template <bool XH>
struct XStage {
  using type = float;
  static __device__ __forceinline__ float put(float v) { return v; }
  static __device__ __forceinline__ float get(float v) { return v; }
};
template <>
struct XStage<true> {
  using type = uint16_t;
  static __device__ __forceinline__ uint16_t put(float v) { return (uint16_t)(__float_as_uint(v) >> 16); }
  static __device__ __forceinline__ float get(uint16_t v) { return __uint_as_float((uint32_t)v << 16); }
};

// MX = false: fields of 16-T bits, the leading bits of the bf16 word.  MX = true: fields of
// 9-T bits (sign, 8-T leading magnitude bits) and one shared exponent per bitmap word: the
// products of a word are summed unscaled and multiplied once by 2^(E + T - 134).  The signed
// magnitude of a field comes from a table of 2^(9-T) floats in LDS, indexed with the field itself: two
// operations and a gather, where taking it apart and converting it took five in a kernel that is
// bound by them (8B shape, mean of the launches of a pass: 22.8 us, now 19.9 with the exponents read through a
// descriptor as well).  The table of a small T is long enough for gathers of a wave to meet in a bank, which eats
// some of the gain but not all: 28672 x 4096 33.1 -> 30.4 us at T = 0 (2.3 conflict cycles per LDS instruction),
// 33.6 -> 28.7 at T = 2 (1.6), 33.6 -> 28.0 at T = 4 (none); 4096 x 4096 7.1 -> 7.1, 6.6, 6.5.
template <int T, int NB, bool MX, bool XH, int FAR = 0>
__global__ __launch_bounds__(kGemvThreads) void gemv_draft_kernel(GemvArgs a) {
  constexpr int FW = MX ? 9 - T : 16 - T;
  using XS = XStage<XH>;
  using XT = typename XS::type;
  static_assert(FAR == 0 || (FAR <= 2 && NB == 1 && !XH), "one column as fp32, a chunk for each item in flight");
  extern __shared__ __attribute__((aligned(16))) uint8_t xs_raw[];
  // shared-exponent form: the table of signed magnitudes in front of x
  uint8_t* const mag_tab = xs_raw + (FAR ? kFarTab : 0);
  XT* xs = reinterpret_cast<XT*>(xs_raw + (MX && !FAR ? kMagTabBytes<FW> : 0));
  const int tid = threadIdx.x;
  const int nchunk = (a.bw + 63) >> 6;
  const int nseg = nchunk * 64;
  const int lane = tid & 63;
  // wave-uniform values are made scalar explicitly so the row/chunk bookkeeping runs on the SALU
  // rows (row pairs) are dealt round-robin to the waves, numbered so that consecutive units go
  // to consecutive workgroups: every workgroup, and every SIMD inside it, gets the same count
  // within one
  const int gw = __builtin_amdgcn_readfirstlane(tid >> 6) * gridDim.x + blockIdx.x;
  const int nwaves = a.nwaves;
  const int pair = a.epi == 2;
  const int row_first = pair ? 2 * gw : gw;
  const bool idle = row_first >= a.rows;  // still helps staging x

  // bitmap words come through a buffer descriptor of the row's words: a word index past the row's
  // end, or a row past the matrix (no records), reads as 0 without a branch
  auto load_bm = [&](const Cursor& c) -> uint32_t {
    const int row = c.row < a.rows ? c.row : 0;
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(a.bitmap + (size_t)row * a.bw), 0, c.row < a.rows ? a.bw * 4 : 0, kRawBufferFlags);
    return __builtin_amdgcn_raw_buffer_load_b32(rs, (c.chunk * 64 + lane) * 4, 0, 0);
  };
  uint32_t rowprefix = 0;  // kept values of the row before the chunk being issued
  auto issue = [&](const Cursor& c, uint32_t m, Window<FW>& w) {
    w.m = m;
    int cnt = __popc(m);
    int incl = wave_incl_scan(cnt);
    int total = __builtin_amdgcn_readlane(incl, 63);
    uint32_t p = rowprefix + (uint32_t)(incl - cnt);
    rowprefix = (c.chunk == nchunk - 1) ? 0u : rowprefix + (uint32_t)total;
    uint32_t bit = __umul24(p, FW);  // p < 2^20: one full-rate multiply
    w.sh = bit & 31u;
    int row = c.row < a.rows ? c.row : row_first;  // past the end: any valid row, its bitmap word is 0
    // The window is read through a buffer descriptor of the row's own part of the stream: words past
    // the row's end read as 0 (range check per word), so a lane that has run out of kept values
    // forms its leftover products from fields of this row or from zeros, never from misaligned bits
    // of the next row (which could look like Inf or NaN and turn 0 * f into NaN).
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(a.spec + (size_t)row * a.sw), 0, a.sw * 4, kRawBufferFlags);
    const int voff = (int)(bit >> 5) * 4;
#pragma unroll
    for (int j = 0; j + 4 <= FW + 1; j += 4) {
      const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rs, voff + 4 * j, 0, 0);
      w.d[j] = v.x; w.d[j + 1] = v.y; w.d[j + 2] = v.z; w.d[j + 3] = v.w;
    }
#pragma unroll
    for (int j = (FW + 1) & ~3; j <= FW; ++j) w.d[j] = __builtin_amdgcn_raw_buffer_load_b32(rs, voff + 4 * j, 0, 0);
    if constexpr (MX) {
      const __amdgpu_buffer_rsrc_t re = __builtin_amdgcn_make_buffer_rsrc(
          (void*)(a.sexp + (size_t)row * a.ew), 0, a.bw, kRawBufferFlags);  // a byte past the row's words reads as 0
      w.e = __builtin_amdgcn_raw_buffer_load_b8(re, c.chunk * 64 + lane, 0, 0);
    }
  };

  float acc[NB], gate[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) acc[b] = gate[b] = 0.f;

  // ITEM: which of the two items in flight
  auto compute = [&](auto ITEM, const Cursor& c, const Window<FW>& w) {
    uint32_t win[FW];
#pragma unroll
    for (int j = 0; j < FW; ++j) win[j] = __builtin_amdgcn_alignbit(w.d[j + 1], w.d[j], w.sh);
    uint32_t m = w.m;
    const XT* xb = xs + ((c.chunk * kXRows + 1) * 64 + lane) * NB;
    uint32_t far[kFarAhead];
    if constexpr (FAR > 0) {
#pragma unroll
      for (int k = 0; k < kFarAhead; ++k) far[k] = (uint32_t)(lane * 4);
    }
    float accw[NB];  // shared-exponent form: unscaled sum of the lane's word
#pragma unroll
    for (int b = 0; b < NB; ++b) accw[b] = 0.f;
    // a step, value I of the lane's word: the reads from LDS (xv: x at its position, fv: the magnitude of the shared-exponent
    // form), then the product
    auto fetch = [&](auto I, float (&xv)[NB], float& fv) {
      constexpr int i = decltype(I)::value;
      if constexpr (FAR > 0) {
        put_lowest_bit(far[i % kFarAhead], m);
        m = drop_lowest(m);
        constexpr int chunk = FAR == 2 ? decltype(ITEM)::value : 0;
        xv[0] = ((const __attribute__((address_space(3))) float*)(uintptr_t)far[i % kFarAhead])[far_row(chunk, 0)];
      } else {
        const XT* xp = xb + lowest_bit(m) * (64 * NB);
        m = drop_lowest(m);
        if constexpr (!XH && (NB == 2 || NB == 4)) {  // two or four columns with one read
          typedef float xvec __attribute__((ext_vector_type(NB)));
          const xvec v = *reinterpret_cast<const xvec*>(xp);
#pragma unroll
          for (int b = 0; b < NB; ++b) xv[b] = v[b];
        } else {
#pragma unroll
          for (int b = 0; b < NB; ++b) xv[b] = XS::get(xp[b]);
        }
      }
      // the field is the index of its signed magnitude; a lane past its last field reads neighbouring
      // bits, always the index of a finite number, and multiplies it by the zero entry of the segment
      if constexpr (MX) fv = *reinterpret_cast<const float*>(mag_tab + field_scaled<FW, i, 2>(win));
    };
    auto use = [&](auto I, const float (&xv)[NB], float fv) {
      constexpr int i = decltype(I)::value;
      if constexpr (MX) {
#pragma unroll
        for (int b = 0; b < NB; ++b) accw[b] = fmaf(fv, xv[b], accw[b]);
      } else {
        const float f = __uint_as_float(field_top<FW, i>(win));
#pragma unroll
        for (int b = 0; b < NB; ++b) acc[b] = fmaf(f, xv[b], acc[b]);
      }
    };
    auto step = [&](auto I) {
      float xv[NB], fv = 0.f;
      fetch(I, xv, fv);
      use(I, xv, fv);
    };
    // the first 16 set bits unconditionally, then pairs until every lane has run out
    if constexpr (FAR > 0) {
      float xv[16][NB], fv[16] = {};
      static_for<0, 16 + kFarAhead>([&](auto I) {
        constexpr int i = decltype(I)::value, done = i - kFarAhead;
        if constexpr (i < 16) fetch(I, xv[i], fv[i]);
        if constexpr (done >= 0) {
          __builtin_amdgcn_sched_barrier(0);
          use(std::integral_constant<int, done>{}, xv[done], fv[done]);
        }
      });
    } else {
      static_for<0, 16>(step);
    }
    auto tail = [&](auto self, auto I) -> void {
      constexpr int i = decltype(I)::value;
      if constexpr (i < 32) {
        if (__builtin_amdgcn_ballot_w64(m != 0u)) {
          std::integral_constant<int, i + 1> I1;
          if constexpr (FAR > 0) {
            float xv[2][NB], fv[2] = {};
            fetch(I, xv[0], fv[0]);
            fetch(I1, xv[1], fv[1]);
            __builtin_amdgcn_sched_barrier(0);
            use(I, xv[0], fv[0]);
            use(I1, xv[1], fv[1]);
          } else {
            step(I);
            step(I1);
          }
          self(self, std::integral_constant<int, i + 2>{});
        }
      }
    };
    tail(tail, std::integral_constant<int, 16>{});
    if constexpr (MX) {
      const float scale = ldexpf(1.0f, (int)w.e + T - 134);
#pragma unroll
      for (int b = 0; b < NB; ++b) acc[b] = fmaf(accw[b], scale, acc[b]);
    }
    if (c.chunk == nchunk - 1) {
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        float s = wave_sum(acc[b]);
        acc[b] = 0.f;
        if (a.epi == 0) {
          if (lane == 0) a.y[(size_t)b * a.yld + c.row] = s;
        } else if (a.epi == 1) {
          uint16_t* hp = a.out16 + (size_t)b * a.yld + c.row;
          if (lane == 0) *hp = f32_to_bf16(bf16_to_f32(*hp) + round_bf16(s));
        } else {
          if (c.row & 1) {  // up row: the gate row came just before
            const float g = round_bf16(gate[b]), u = round_bf16(s);
            if (lane == 0) a.out16[(size_t)b * (a.yld >> 1) + (c.row >> 1)] = f32_to_bf16(g / (1.0f + expf(-g)) * u);
          } else {
            gate[b] = s;
          }
        }
      }
    }
  };

  // ---- x is staged in blocks [chunk][1 + 32][64][NB]; row 0 of a block is 0.0.
  // Fast path (cols a multiple of 8, at most 2 pieces of 8 per thread): x and the norm gain are
  // read once with 16-byte loads, requested before anything else so they travel together with
  // the first bitmap words, and stay in registers between the norm reduction and the LDS writes.
  const int npiece = (nseg * 32) >> 3;  // pieces of 8 columns, including the zero tail
  const bool fast = (a.cols & 7) == 0 && npiece <= 2 * kGemvThreads &&
                    ((reinterpret_cast<uintptr_t>(a.x) | reinterpret_cast<uintptr_t>(a.gain)) & 15) == 0;
  uint4 raw[2][NB], gv[2];
  auto stage_load = [&]() {
    if (!fast) return;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int col = (tid + k * kGemvThreads) * 8;
      gv[k] = make_uint4(0, 0, 0, 0);
      if (a.gain && col < a.cols) gv[k] = *reinterpret_cast<const uint4*>(a.gain + col);
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        raw[k][b] = make_uint4(0, 0, 0, 0);
        if (col < a.cols) raw[k][b] = *reinterpret_cast<const uint4*>(a.x + (size_t)b * a.cols + col);
      }
    }
  };
  auto stage_x = [&]() {
    if constexpr (MX) {
      if (tid < (1 << FW)) {
        const float mag = (float)(tid & ((1 << (FW - 1)) - 1));
        reinterpret_cast<float*>(mag_tab)[tid] = (tid >> (FW - 1)) ? -mag : mag;
      }
    }
    if constexpr (FAR > 0) {
      for (int sgi = tid; sgi < nseg; sgi += kGemvThreads) xs[far_row(sgi >> 6, 255) + (sgi & 63)] = 0.f;
    }
    for (int sgi = tid; sgi < (FAR ? 0 : nseg); sgi += kGemvThreads) {
#pragma unroll
      for (int b = 0; b < NB; ++b) xs[(((sgi >> 6) * kXRows) * 64 + (sgi & 63)) * NB + b] = XS::put(0.f);
    }
    float rn[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) rn[b] = 1.f;
    float* red;  // [NB][kGemvWaves]
    if constexpr (FAR > 0) {
      red = reinterpret_cast<float*>(xs_raw + kFarRed);
    } else {
      __shared__ float red_[NB * kGemvWaves];
      red = red_;
    }
    auto finish_norm = [&](const float (&ss)[NB]) {
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        float t = wave_sum(ss[b]);
        if (lane == 0) red[b * kGemvWaves + (tid >> 6)] = t;
      }
      __syncthreads();
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        float t = 0.f;
#pragma unroll
        for (int w = 0; w < kGemvWaves; ++w) t += red[b * kGemvWaves + w];
        rn[b] = 1.0f / sqrtf(t / (float)a.cols + a.eps);
      }
    };
    if (fast) {
      if (a.gain) {
        float ss[NB];
#pragma unroll
        for (int b = 0; b < NB; ++b) {
          ss[b] = 0.f;
#pragma unroll
          for (int k = 0; k < 2; ++k) {
            const uint32_t wd[4] = {raw[k][b].x, raw[k][b].y, raw[k][b].z, raw[k][b].w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              float lo = __uint_as_float(wd[e] << 16), hi = __uint_as_float(wd[e] & 0xFFFF0000u);
              ss[b] += lo * lo;
              ss[b] += hi * hi;
            }
          }
        }
        finish_norm(ss);
      }
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const int piece = tid + k * kGemvThreads;
        const int col = piece * 8;
        if (piece < npiece) {
          const uint32_t gw4[4] = {gv[k].x, gv[k].y, gv[k].z, gv[k].w};
          XT* dst = xs + (FAR ? far_index(col) : x_index<NB>(col));  // the 8 columns of a piece lie in one word: 64 * NB apart
#pragma unroll
          for (int b = 0; b < NB; ++b) {
            const uint32_t wd[4] = {raw[k][b].x, raw[k][b].y, raw[k][b].z, raw[k][b].w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              float lo = __uint_as_float(wd[e] << 16), hi = __uint_as_float(wd[e] & 0xFFFF0000u);
              if (a.gain) {
                lo = round_bf16(lo * rn[b] * __uint_as_float(gw4[e] << 16));
                hi = round_bf16(hi * rn[b] * __uint_as_float(gw4[e] & 0xFFFF0000u));
              }
              dst[(2 * e) * 64 * NB + b] = XS::put(lo);
              dst[(2 * e + 1) * 64 * NB + b] = XS::put(hi);
            }
          }
        }
      }
    } else {
      if (a.gain) {
        float ss[NB];
#pragma unroll
        for (int b = 0; b < NB; ++b) {
          ss[b] = 0.f;
          for (int c = tid; c < a.cols; c += kGemvThreads) {
            float v = bf16_to_f32(a.x[(size_t)b * a.cols + c]);
            ss[b] += v * v;
          }
        }
        finish_norm(ss);
      }
      for (int col = tid; col < nseg * 32; col += kGemvThreads) {
#pragma unroll
        for (int b = 0; b < NB; ++b) {
          float v = 0.f;
          if (col < a.cols) {
            v = bf16_to_f32(a.x[(size_t)b * a.cols + col]);
            if (a.gain) v = round_bf16(v * rn[b] * bf16_to_f32(a.gain[col]));
          }
          xs[(FAR ? far_index(col) : x_index<NB>(col)) + b] = XS::put(v);
        }
      }
    }
    __syncthreads();
  };
  Cursor cb{row_first, 0}, ci{row_first, 0}, cc{row_first, 0};
  Window<FW> w0, w1;
  stage_load();
  if (idle) {
    stage_x();
    return;
  }
  uint32_t m0 = load_bm(cb); cb.advance(nchunk, nwaves, pair);
  uint32_t m1 = load_bm(cb); cb.advance(nchunk, nwaves, pair);
  issue(ci, m0, w0); ci.advance(nchunk, nwaves, pair);
  stage_x();  // overlaps the first bitmap and window loads
  while (true) {
    uint32_t m2 = load_bm(cb); cb.advance(nchunk, nwaves, pair);
    issue(ci, m1, w1); ci.advance(nchunk, nwaves, pair);
    compute(std::integral_constant<int, 0>{}, cc, w0); cc.advance(nchunk, nwaves, pair);
    if (cc.row >= a.rows) break;
    m1 = load_bm(cb); cb.advance(nchunk, nwaves, pair);
    issue(ci, m2, w0); ci.advance(nchunk, nwaves, pair);
    compute(std::integral_constant<int, 1>{}, cc, w1); cc.advance(nchunk, nwaves, pair);
    if (cc.row >= a.rows) break;
  }
}

// LDS allowance of the instantiation, then the launch
template <int T, int NB, bool MX, bool XH, int FAR = 0>
static int launch_gemv_instance(cas_ctx* ctx, const GemvArgs& a, int grid, size_t lds) {
  static LdsLimit lim;
  const int rc = allow_lds(ctx, (const void*)gemv_draft_kernel<T, NB, MX, XH, FAR>, lds, lim, FAR > 0);
  if (rc != CAS_OK) return rc;
  hipLaunchKernelGGL((gemv_draft_kernel<T, NB, MX, XH, FAR>), dim3(grid), dim3(kGemvThreads), lds, ctx->stream, a);
  CAS_HIP(ctx, hipGetLastError());
  return CAS_OK;
}

// Chunks of the form with x far apart, 0 where it does not take the rows, and its LDS bytes: 64 KB, and 8 for a second chunk,
// so that two workgroups, of two streams, share a CU.  With 64 KB per chunk they did not.  us a product, two / three streams with
// a chain of them each, 64 KB per chunk / now / the form with x side by side: 4096 x 4096 5.4 / 5.1 / 5.3, 5.5 / 4.5 / 4.7; 28672
// x 4096 24.2 / 21.9 / 22.8, 24.8 / 21.5 / 22.9, over shared exponents 23.9 / 17.9 / 20.2, 25.0 / 19.6 / 21.3; 1024 x 1024 2.85 /
// 2.83 / 2.89, 2.15 / 2.13 / 2.18; one stream 26.3 / 26.5 / 28.4 (28672 x 4096).  More than two chunks would need as many items of a
// wave in flight, or an operation for the address.
static inline size_t gemv_far_bytes(int chunks) { return kFarZero + (size_t)(chunks - 1) * kFarChunk; }
static inline int gemv_far_chunks(const cas_ctx* ctx, int bw) {
  const int chunks = (bw + 63) / 64;
  return chunks <= 2 && gemv_far_bytes(2) <= (size_t)ctx->lds_max ? chunks : 0;
}

// LDS bytes of the staged x
static inline size_t gemv_lds_bytes(int bw, int batch, bool half) {
  return (half ? sizeof(uint16_t) : sizeof(float)) * (size_t)((bw + 63) / 64 * 64) * kXRows * batch;
}

// One workgroup per CU (16 waves), or one per row (gate/up row pair) of a matrix that has fewer: every workgroup stages x
// once.  Two per CU for every matrix took a 28672 x 4096 product alone from 28.8 to
// 26.9 us in the form with x side by side, but rounds from 19.9 to 20.2 ms and from 8.35 to 9.05 with four columns.
static inline int gemv_grid(const cas_ctx* ctx, int64_t units) { return (int)std::min<int64_t>(ctx->num_cu, units); }

}  // namespace cas
