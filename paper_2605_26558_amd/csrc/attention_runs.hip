// Attention over runs of columns (attention.hip), exact form: up to 64 query rows of a run per kv head.
#include "attention_kernel.inl"

namespace cas {
template int launch_mt<1, true, false>(cas_ctx*, const AttnRuns&, dim3);
template int launch_mt<2, true, false>(cas_ctx*, const AttnRuns&, dim3);
template int launch_mt<3, true, false>(cas_ctx*, const AttnRuns&, dim3);
template int launch_mt<4, true, false>(cas_ctx*, const AttnRuns&, dim3);
}  // namespace cas
