// Attention over runs of columns (attention.hip), exact form over a cache with shared exponents: the length of a run is
// given there, up to 80 query rows per kv head.
#include "attention_kernel.inl"

namespace cas {
template int launch_mt<1, true, true>(cas_ctx*, const AttnRuns&, dim3);
template int launch_mt<2, true, true>(cas_ctx*, const AttnRuns&, dim3);
template int launch_mt<3, true, true>(cas_ctx*, const AttnRuns&, dim3);
template int launch_mt<4, true, true>(cas_ctx*, const AttnRuns&, dim3);
template int launch_mt<5, true, true>(cas_ctx*, const AttnRuns&, dim3);
}  // namespace cas
