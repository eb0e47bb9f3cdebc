// Prefill attention of small plans: the instantiations of the kernels in kvx_attn_kernels.h
// that take their units from the kernel arguments.  In a file of their own, as the mixed
// ones are: this leaves the code of the plain kernels alone, whose main loop has no scalar
// register to spare.  Such a call is one launch, without a copy or a kernel that writes the
// units before it.  us per call with units copied / written by a kernel / here: 4 requests of
// 8 to 100 tokens on 4/2/64 heads 21.5 / 17.5 / 11.9; 12 of 20 to 700 on 8/2/64 heads
// 72 / 49 / 41; 6 of 275 to 1163 on 8/2/64 heads 55 / 49 / 38.7.  The main loop is as good
// as the plain one's (983 instructions against 979), so every compact plan takes this path:
// 2 requests of 512 tokens on 131072 each, 907 us here and 906 in the plain kernel.

#include "kvx_attn_kernels.h"

namespace kvx {

static_assert(sizeof(AttnParams) % 8 == 0 && sizeof(AttnParams) + sizeof(CompactPlan) <= 4096, "kernel arguments");

hipError_t launch_small_attention(const AttnParams& p, int64_t n_units, int head_dim, bool fp8, bool scaled_q,
                                  hipStream_t stream) {
  launch_attn<false>(p, *p.compact, n_units, head_dim, fp8, scaled_q, stream);
  return hipGetLastError();
}

}  // namespace kvx
