// Prefill attention: the launches of the kernels in kvx_attn_kernels.h for batches without
// decode units, and the merge of split parts.

#include "kvx_attn_kernels.h"

namespace kvx {
namespace {

// Combine the parts of split tiles: o = sum_p e^{lse_p - M} o_p / sum_p e^{lse_p - M}.
// Workgroup (merge, 32-row block, 32 dims b): wave g4 combines dims 32 b + 8 g4 .. +8 of
// the block, lane by lane in the layout write_result stores, with the loads of UNROLL
// parts in flight.  256 parts of 256 rows (33.5 MB): 7.6 us, against 17.9 us for a serial
// loop over parts in row order.
template <int D>
__global__ __launch_bounds__(256) void merge_kernel(MergeParams p) {
  constexpr int UNROLL = 8;
  constexpr int DB = Geom<D>::DB;
  MergeUnit mu;
  if (p.plan.n > 0) {
    const int h = blockIdx.x % p.plan.heads;
    mu = p.plan.merge[blockIdx.x / p.plan.heads];
    mu.head_ntok += h << 16;
    mu.part0 += h * mu.nparts;
  } else {
    mu = p.merges[blockIdx.x];
  }
  const int kv_head = mu.head_ntok >> 16;
  const int ntok = mu.head_ntok & 0xFFFF;
  const int blk = (int)blockIdx.y / DB, b = (int)blockIdx.y % DB;
  const int lane = threadIdx.x & 63, g4 = threadIdx.x >> 6;
  const int rho = blk * 32 + (lane & 31);
  const int tok = rho / p.group;
  if (tok >= ntok) return;
  const float* lse = p.lse_part + (size_t)mu.part0 * kTileRows + rho;
  const float* op = p.o_part + (size_t)mu.part0 * kTileRows * D + blk * (32 * D) + (4 * b + g4) * 256 + lane * 4;
  float mx = -INFINITY, wsum = 0.0f;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  for (int q0 = 0; q0 < mu.nparts; q0 += UNROLL) {
    float l[UNROLL];
    f32x4 x[UNROLL];
    float m_new = mx;
#pragma unroll
    for (int j = 0; j < UNROLL; j++) {
      const bool in = q0 + j < mu.nparts;
      l[j] = in ? lse[(size_t)(q0 + j) * kTileRows] : -INFINITY;
      x[j] = in ? *(const f32x4*)(op + (size_t)(q0 + j) * kTileRows * D) : f32x4{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int j = 0; j < UNROLL; j++) m_new = fmaxf(m_new, l[j]);
    const float alpha = mx == -INFINITY ? 0.0f : __expf(mx - m_new);
    wsum *= alpha;
    acc *= alpha;
#pragma unroll
    for (int j = 0; j < UNROLL; j++) {
      const float w = (l[j] == -INFINITY) ? 0.0f : __expf(l[j] - m_new);
      acc += x[j] * w;
      wsum += w;
    }
    mx = m_new;
  }
  const float inv = wsum > 0.0f ? 1.0f / wsum : 0.0f;
  const int hq = kv_head * p.group + (rho - tok * p.group);
  const size_t row = (size_t)(mu.qo_row0 + tok) * p.num_q_heads + hq;
  uint2 w2;
  w2.x = pack_bf16(acc[0] * inv, acc[1] * inv);
  w2.y = pack_bf16(acc[2] * inv, acc[3] * inv);
  *(uint2*)(p.out + row * D + 32 * b + 8 * g4 + 4 * (lane >> 5)) = w2;
  if (p.lse != nullptr && b == 0 && g4 == 0 && lane < 32) p.lse[row] = mx + __logf(wsum);
}

}  // namespace

hipError_t launch_extend_attention(const AttnParams& p, int64_t n_units, int head_dim, bool fp8, bool scaled_q,
                                   hipStream_t stream) {
  if (n_units <= 0) return hipSuccess;
  if (p.compact != nullptr) return launch_small_attention(p, n_units, head_dim, fp8, scaled_q, stream);
  if (p.mixed) return launch_mixed_attention(p, n_units, head_dim, fp8, scaled_q, stream);
  launch_attn<false>(p, UnitsInMemory{}, n_units, head_dim, fp8, scaled_q, stream);
  return hipGetLastError();
}

hipError_t launch_merge(const MergeParams& p, int64_t n_merges, int head_dim, hipStream_t stream) {
  if (n_merges <= 0) return hipSuccess;
  const dim3 block(256);
  if (head_dim == 128)
    hipLaunchKernelGGL((merge_kernel<128>), dim3((unsigned)n_merges, kTileRows / 32 * Geom<128>::DB), block, 0, stream, p);
  else
    hipLaunchKernelGGL((merge_kernel<64>), dim3((unsigned)n_merges, kTileRows / 32 * Geom<64>::DB), block, 0, stream, p);
  return hipGetLastError();
}

}  // namespace kvx
