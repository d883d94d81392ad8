// Attention over runs of columns (attention.hip), exact form: up to 64 query rows of a run per kv head, and up to 80
// where the run is given (a cache with shared exponents).
#include "attention_kernel.inl"

namespace cas {
template int launch_mt<4, true, false>(cas_ctx*, const AttnRuns&, dim3);
template int launch_mt<4, true, true>(cas_ctx*, const AttnRuns&, dim3);
template int launch_mt<5, true, true>(cas_ctx*, const AttnRuns&, dim3);
}  // namespace cas
