// Prefill attention of batches that mix prefill with one-token suffixes: the MIXED
// instantiations of the kernels in kvx_attn_kernels.h.  In a file of their own: next to
// them, the compiler simplifies the helpers both use in another order, and the plain
// bf16 kernel came out 9% slower.

#include "kvx_attn_kernels.h"

namespace kvx {

hipError_t launch_mixed_attention(const AttnParams& p, int64_t n_units, int head_dim, bool fp8, bool scaled_q,
                                  hipStream_t stream) {
  launch_attn<true>(p, UnitsInMemory{}, n_units, head_dim, fp8, scaled_q, stream);
  return hipGetLastError();
}

}  // namespace kvx
