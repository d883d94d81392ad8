// Draft GEMV: y = Wdraft x, reading only the speculation data (bitmap + spec stream) and
// decoding it inside the kernel (Sec. 4.1 draft inference: zero padding of pruned positions
// and dropped mantissa bits).
//
// Mapping.  One wave walks one output row at a time in chunks of 64 bitmap words (2048
// columns): lane l owns word l of the chunk, i.e. 32 consecutive columns.  A DPP prefix sum of
// the popcounts gives each lane the index of its first kept value, so its fields are one
// contiguous run of the row's spec stream; neighbouring lanes read neighbouring runs.  The
// lane loads a window of 16-t+1 words at its run, aligns it with funnel shifts, and then
// walks the set bits of its word: field i of the window belongs to the i-th set bit.  Placing
// a field at the top of a 32-bit register yields the fp32 value of the zero-padded bf16.
// x sits in LDS as fp32 in segments of 1+32 entries per bitmap word; entry 0 of a segment is
// 0.0, so a lane that has run out of set bits (bit position -1) multiplies by zero (one column of up to 4096 values:
// 256 bytes from position to position, FAR in the kernel).
// The (row, chunk) items of a wave run through a three-stage software pipeline: bitmap word of
// item q+2, prefix + window loads of item q+1, arithmetic of item q.
#include "gemv_draft_kernel.inl"

namespace cas {

// A batch takes x as fp32 where that fits (2 columns to 18432 values each, 3 to 12288, 4 to 8192): it is the faster
// form at every size measured (XStage); wider rows keep to bf16.
template <int T, int NB>
static int launch_nb(cas_ctx* ctx, const GemvArgs& a, int grid) {
  if constexpr (NB == 1) {
    const int far = gemv_far_chunks(ctx, a.bw);
    if (far == 1) return launch_gemv_instance<T, 1, false, false, 1>(ctx, a, grid, gemv_far_bytes(1));
    if (far == 2) return launch_gemv_instance<T, 1, false, false, 2>(ctx, a, grid, gemv_far_bytes(2));
  }
  const size_t lds = gemv_lds_bytes(a.bw, NB, false);
  if (lds <= (size_t)ctx->lds_max) return launch_gemv_instance<T, NB, false, false>(ctx, a, grid, lds);
  if constexpr (NB > 1) return launch_gemv_instance<T, NB, false, true>(ctx, a, grid, gemv_lds_bytes(a.bw, NB, true));
  return CAS_ENOTSUP;
}

template <int T>
static int launch_t(cas_ctx* ctx, const GemvArgs& a, int batch, int grid) {
  switch (batch) {
    case 1: return launch_nb<T, 1>(ctx, a, grid);
    case 2: return launch_nb<T, 2>(ctx, a, grid);
    case 3: return launch_nb<T, 3>(ctx, a, grid);
    case 4: return launch_nb<T, 4>(ctx, a, grid);
    default: return CAS_EINVAL;
  }
}

int launch_gemv_draft(cas_ctx* ctx, const cas_wdesc& d, const void* spec, const uint16_t* x, int batch, float* y) {
  return launch_gemv_draft_fused(ctx, d, spec, x, batch, y, nullptr, 0.f, 0, nullptr);
}

int launch_gemv_draft_block(cas_ctx* ctx, const cas_wdesc& d, const uint32_t* bitmap, const uint32_t* spec, int nr,
                            const uint16_t* x, int batch, float* y, const uint16_t* gain, float eps, int epi,
                            uint16_t* out16) {
  GemvArgs a{};
  a.gain = gain; a.eps = eps; a.epi = epi; a.out16 = out16;
  a.rows = nr; a.cols = (int)d.cols; a.bw = d.bw; a.sw = d.sw;
  a.bitmap = bitmap;
  a.spec = spec;
  a.x = x; a.y = y; a.yld = (int)d.rows;
  if (gemv_lds_bytes(d.bw, batch, batch > 1) > (size_t)ctx->lds_max) return CAS_ENOTSUP;
  const int grid = gemv_grid(ctx, epi == 2 ? nr / 2 : nr);  // a gate/up row pair stays in one wave
  a.nwaves = grid * kGemvWaves;
#define CAS_T(TV) case TV: return launch_t<TV>(ctx, a, batch, grid);
  switch (d.t) {
    CAS_T(0) CAS_T(1) CAS_T(2) CAS_T(3) CAS_T(4) CAS_T(5) CAS_T(6) CAS_T(7)
  }
#undef CAS_T
  return CAS_EINVAL;
}

int launch_gemv_draft_fused(cas_ctx* ctx, const cas_wdesc& d, const void* spec, const uint16_t* x, int batch,
                            float* y, const uint16_t* gain, float eps, int epi, uint16_t* out16) {
  if (d.rows <= 0) return CAS_OK;
  if (epi == 2 && (d.rows & 1)) return CAS_EINVAL;
  if (gemv_lds_bytes(d.bw, batch, batch > 1) > (size_t)ctx->lds_max) return CAS_ENOTSUP;
  ProfScope prof(ctx, PROF_GEMV_DRAFT, 4.0 * (double)d.rows * (d.bw + d.sw));
  return launch_gemv_draft_block(ctx, d, (const uint32_t*)((const char*)spec + d.off_bitmap),
                                 (const uint32_t*)((const char*)spec + d.off_spec), (int)d.rows, x, batch, y, gain, eps,
                                 epi, out16);
}

}  // namespace cas
