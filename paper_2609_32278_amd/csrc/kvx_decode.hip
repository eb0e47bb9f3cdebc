// Paged decode attention over the KV pool, gfx950 (CDNA4): one new token per
// request attends over the request's whole cached sequence (the decode step that
// follows prefill, paper Section 2 and Section 4's prefill-decode serving).
//
// A decode step reads every K/V byte of a request once for a handful of query
// rows (the G query heads of one KV head), so it is bound by HBM, not MFMA.  The
// kernel streams pages straight into registers with wide loads and keeps several
// page pairs in flight per wave:
//   * workgroup = one key chunk of one (request, KV head); 4 waves, wave w takes
//     page pairs w, w+4, w+8, ... of the chunk (two 16-key pages = 32 keys);
//   * S^T (16 keys x 16 rows) = K Q^T on v_mfma_f32_16x16x32_bf16: the page's keys
//     are the A operand straight from global memory, the G <= 16 query heads the B
//     operand (rows past G are zero);
//   * softmax in base 2, exact online rescaling (a row's four lane groups share
//     its running maximum through two lane swaps);
//   * O^T (16 dims x 16 rows per block) += V^T P^T, again 16x16x32: the 32 keys of
//     the pair are the reduction dimension, taken as key 4g..4g+3 of the first
//     page and of the second page in lane group g -- the keys that lane group
//     holds in the S^T result, so P needs no data movement between lanes;
//   * the four waves' partial results are combined through LDS; a chunk that is
//     one part of a split key range writes (O, LSE), merged afterwards.

#include "kvx_decode_unit.h"

namespace kvx {
namespace {

using decode::f32x4;
using decode::kRows;
using decode::pack2;

constexpr int kWaves = kDecodeThreads / 64;

// The work item of this workgroup (scalar loads: everything derived stays uniform).
__device__ __forceinline__ DecodeUnit unit_of(const DecodeParams& p) {
  using decode::const_i32_ptr;
  const_i32_ptr w = (const_i32_ptr)(p.units + blockIdx.x);
  int h = 0;
  if (p.plan.n > 0) {  // in the kernel arguments
    w = (const_i32_ptr)((const __attribute__((address_space(4))) char*)__builtin_amdgcn_kernarg_segment_ptr() +
                        offsetof(DecodeParams, plan.unit)) +
        (blockIdx.x / p.plan.heads) * (sizeof(DecodeUnit) / 4);
    h = blockIdx.x % p.plan.heads;
  }
  DecodeUnit u;
  u.qo_row = w[0];
  u.page_base = w[1];
  u.key_begin = w[2];
  u.key_end = w[3];
  u.head = w[4] + h;
  u.part = w[5] < 0 ? -1 : w[5] + h * w[6];
  return u;
}

// Whether another request's page list holds this chunk's first page at the same place
// (prefixes are shared in whole pages from the start).  Uniform; at most four lists per lane.
__device__ __forceinline__ bool chunk_is_shared(const DecodeParams& p, const DecodeUnit& u) {
  const int32_t* base = p.lists.base;
  if (base == nullptr)
    base = (const int32_t*)((const __attribute__((address_space(4))) char*)__builtin_amdgcn_kernarg_segment_ptr() +
                            offsetof(DecodeParams, lists.in_args));
  const int lp = u.key_begin / kPageSize, own = ((decode::const_i32_ptr)p.a.page_ids)[u.page_base + lp];
  bool same = false;
#pragma unroll
  for (int j = 0; j < kShareReqs / 64; j++) {
    const int i = (threadIdx.x & 63) + 64 * j;
    if (i >= p.lists.n) continue;
    const int b = base[i];
    if (b != u.page_base && lp < base[i + 1] - b) same |= p.a.page_ids[b + lp] == own;
  }
  return __any(same);
}

// NT: a chunk whose pages one request alone holds is read with non-temporal loads, which
// spares the caches for the others; pages of a shared prefix are read again by every request
// that holds them, mostly out of the XCD's L2, and keep plain loads.  us per call plain / all
// non-temporal / told apart: 64 agents of 16k private tokens, 32/8/128 heads, 745 / 682 / 667;
// 128 agents on one 16k prefix 718 / 928 / 728, on 16 of them 760 / 1075 / 751, on one of 4k
// with 4k private tokens each 564 / 554 / 523; 128 on one of 64k, fp8 pool, 64/8/128 heads,
// 1176 / 1997 / 1188.
template <int D, bool FP8, bool NT>
__global__ __launch_bounds__(kDecodeThreads, 2) void decode_kernel(DecodeParams p) {
  __shared__ float o[kWaves * kRows * D], m[kWaves * kRows], l[kWaves * kRows];
  const decode::CombineShared<D, kWaves> sm{o, m, l};
  const DecodeUnit u = unit_of(p);
  auto nt = [&]() { return NT && !chunk_is_shared(p, u); };
  if constexpr (FP8) decode::decode_unit_fp8<D, kWaves, false>(p.a, u, sm, nt);
  else decode::decode_unit<D, kWaves, false>(p.a, u, sm, nt);
}

// Combine the parts of a split decode key range: o = sum_p e^{lse_p - M} o_p / sum_p e^{lse_p - M}.
// Latency bound: a merge reads a few KiB per part.  One workgroup per (merge, query
// row): D / 4 lanes hold the row's 16-byte columns, and 256 / (D / 4) lane groups take
// every such part each, so that the parts' loads are in flight together; the groups
// meet in LDS.  One workgroup per merge with a serial loop over the parts took 43 us for
// 192 merges of 3-22 parts (8 rows of 128), this takes 4.3 us.
template <int D>
__global__ __launch_bounds__(256) void decode_merge_kernel(DecodeMergeParams p) {
  constexpr int C4 = D / 4;        // lanes per row
  constexpr int PG = 256 / C4;     // part groups
  constexpr int UNROLL = 4;        // parts in flight per group
  __shared__ float sm_m[PG], sm_w[PG];
  __shared__ f32x4 sm_o[PG][C4];
  DecodeMerge mu;
  if (p.plan.n > 0) {
    const int h = blockIdx.x % p.plan.heads;
    mu = p.plan.merge[blockIdx.x / p.plan.heads];
    mu.head += h;
    mu.part0 += h * mu.nparts;
  } else {
    mu = p.merges[blockIdx.x];
  }
  const int row = blockIdx.y;
  const int c = threadIdx.x % C4, pg = threadIdx.x / C4;
  const float* lse = p.lse_part + (size_t)mu.part0 * kRows + row;
  const float* o = p.o_part + ((size_t)mu.part0 * kRows + row) * D + 4 * c;
  float M = -INFINITY, wsum = 0.f;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  for (int q0 = pg; q0 < mu.nparts; q0 += UNROLL * PG) {
    float l[UNROLL];
    f32x4 x[UNROLL];
    float m_new = M;
#pragma unroll
    for (int j = 0; j < UNROLL; j++) {
      const int q = q0 + j * PG;
      const bool in = q < mu.nparts;
      l[j] = in ? lse[(size_t)q * kRows] : -INFINITY;
      x[j] = in ? *(const f32x4*)(o + (size_t)q * kRows * D) : f32x4{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int j = 0; j < UNROLL; j++) m_new = fmaxf(m_new, l[j]);
    const float alpha = M == -INFINITY ? 0.f : __expf(M - m_new);
    wsum *= alpha;
    acc *= alpha;
#pragma unroll
    for (int j = 0; j < UNROLL; j++) {
      const float w = l[j] == -INFINITY ? 0.f : __expf(l[j] - m_new);
      wsum += w;
      acc += w * x[j];
    }
    M = m_new;
  }
  sm_o[pg][c] = acc;
  if (c == 0) {
    sm_m[pg] = M;
    sm_w[pg] = wsum;
  }
  __syncthreads();
  if (pg != 0) return;
#pragma unroll
  for (int i = 1; i < PG; i++) M = fmaxf(M, sm_m[i]);
  wsum = 0.f;
  acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int i = 0; i < PG; i++) {
    const float e = sm_m[i] == M ? 1.f : __expf(sm_m[i] - M);
    wsum += e * sm_w[i];
    acc += e * sm_o[i][c];
  }
  const float inv = wsum > 0.f ? 1.0f / wsum : 0.f;
  const size_t orow = (size_t)mu.qo_row * p.num_q_heads + mu.head * p.group + row;
  *(uint2*)(p.out + orow * D + 4 * c) = make_uint2(pack2(acc[0] * inv, acc[1] * inv), pack2(acc[2] * inv, acc[3] * inv));
  if (p.lse != nullptr && c == 0) p.lse[orow] = M + __logf(wsum);
}

}  // namespace

template <int D, bool FP8>
static void launch_decode_for(const DecodeParams& p, int64_t n_units, hipStream_t stream) {
  const dim3 grid((unsigned)n_units), block(kDecodeThreads);
  if (p.lists.n > 0) hipLaunchKernelGGL((decode_kernel<D, FP8, true>), grid, block, 0, stream, p);
  else hipLaunchKernelGGL((decode_kernel<D, FP8, false>), grid, block, 0, stream, p);
}

hipError_t launch_decode(const DecodeParams& p, int64_t n_units, int head_dim, bool fp8, hipStream_t stream) {
  if (n_units <= 0) return hipSuccess;
  if (head_dim == 128) {
    if (fp8) launch_decode_for<128, true>(p, n_units, stream);
    else launch_decode_for<128, false>(p, n_units, stream);
  } else {
    if (fp8) launch_decode_for<64, true>(p, n_units, stream);
    else launch_decode_for<64, false>(p, n_units, stream);
  }
  return hipGetLastError();
}

hipError_t launch_decode_merge(const DecodeMergeParams& p, int64_t n_merges, int head_dim, hipStream_t stream) {
  if (n_merges <= 0) return hipSuccess;
  const dim3 grid((unsigned)n_merges, (unsigned)p.group), block(256);
  if (head_dim == 128) hipLaunchKernelGGL(decode_merge_kernel<128>, grid, block, 0, stream, p);
  else hipLaunchKernelGGL(decode_merge_kernel<64>, grid, block, 0, stream, p);
  return hipGetLastError();
}

}  // namespace kvx
