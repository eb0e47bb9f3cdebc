// Device code of a decode unit -- one query token of a request and KV head over a chunk of
// its keys -- shared by the decode kernels and by the prefill kernels of batches that mix
// both.  Included once per .hip file, inside no namespace.
#pragma once

#include <type_traits>

#include "kvx_internal.h"

namespace kvx {
namespace {
namespace decode {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef const __attribute__((address_space(4))) int32_t* const_i32_ptr;  // scalar-loaded

constexpr float kLn2 = 0.6931471805599453f;
constexpr int kRows = kDecodeMaxGroup;

__device__ __forceinline__ uint32_t pack2(float a, float b) {
  bf16x2 v;
  v[0] = (__bf16)a;
  v[1] = (__bf16)b;
  return __builtin_bit_cast(uint32_t, v);
}

// A 16- or 8-byte load of pool data; NT: not kept in the caches (non-temporal).
template <bool NT>
__device__ __forceinline__ uint4 load16(const void* p) {
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  if constexpr (!NT) return *(const uint4*)p;
  return __builtin_bit_cast(uint4, __builtin_nontemporal_load((const u32x4*)p));
}
template <bool NT>
__device__ __forceinline__ uint2 load8(const void* p) {
  typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
  if constexpr (!NT) return *(const uint2*)p;
  return __builtin_bit_cast(uint2, __builtin_nontemporal_load((const u32x2*)p));
}

// max / sum over the four lane groups (lanes n, n+16, n+32, n+48) holding one row
__device__ __forceinline__ float group_max(float x) {
  x = fmaxf(x, __shfl_xor(x, 16));
  return fmaxf(x, __shfl_xor(x, 32));
}
__device__ __forceinline__ float group_sum(float x) {
  x += __shfl_xor(x, 16);
  return x + __shfl_xor(x, 32);
}

// 8 fp8 e4m3 codes -> 8 bf16 (exact: e4m3 values are bf16 values)
__device__ __forceinline__ uint4 fp8x8_bf16(uint2 c) {
  return make_uint4(__builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(c.x, 1.0f, false)),
                    __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(c.x, 1.0f, true)),
                    __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(c.y, 1.0f, false)),
                    __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(c.y, 1.0f, true)));
}

// Shared memory of a workgroup's combine: every wave's O [NW][kRows][D], row maxima and
// sums [NW][kRows] each.
template <int D, int NW>
struct CombineShared {
  float* o;
  float* m;
  float* l;
};

// Combine the waves' partial results through LDS and write the chunk's result.
// Lane (n, g) holds dims 16 b + 4 g + i of row n, relative to its row maximum m_run
// (log2 units), and the part l_run of the row sum over its own keys.  A row whose sum is a
// NaN (a NaN or an infinite score) is written as zeros, and as NaN with NANS, which is
// what a prefill tile gives: one-token requests beside longer ones keep that.  They also
// get a tile's `none` where no score is above -inf: 0, on an fp8 pool NaN.
template <int D, int NW, bool NANS>
__device__ __forceinline__ void combine_waves(const DecodeArgs& p, const DecodeUnit& u, CombineShared<D, NW> sm,
                                              const f32x4 (&o)[D / 16], float m_run, float l_run, float vscale,
                                              float none) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int n = lane & 15, g = lane >> 4, G = p.group;
  const float l_row = group_sum(l_run);
  if (g == 0) {
    sm.m[wave * kRows + n] = m_run;
    sm.l[wave * kRows + n] = l_row;
  }
#pragma unroll
  for (int b = 0; b < D / 16; b++)
#pragma unroll
    for (int i = 0; i < 4; i++) sm.o[(wave * kRows + n) * D + 16 * b + 4 * g + i] = o[b][i];
  __syncthreads();
  for (int idx = threadIdx.x; idx < G * D; idx += 64 * NW) {
    const int row = idx / D, d = idx - row * D;
    float M = -INFINITY;
#pragma unroll
    for (int w = 0; w < NW; w++) M = fmaxf(M, sm.m[w * kRows + row]);
    float wsum = 0.f, acc = 0.f;
    if (NANS || M != -INFINITY) {
#pragma unroll
      for (int w = 0; w < NW; w++) {
        const float e = sm.m[w * kRows + row] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(sm.m[w * kRows + row] - M);
        wsum += e * sm.l[w * kRows + row];
        acc += e * sm.o[(w * kRows + row) * D + d];
      }
    }
    const float val = wsum > 0.f ? acc * vscale / wsum : !NANS ? 0.f : wsum == 0.f ? none : acc * 0.f;
    const float lse_v = wsum > 0.f ? (M + __log2f(wsum)) * kLn2 : -INFINITY;
    if (u.part < 0) {
      const size_t orow = (size_t)u.qo_row * p.num_q_heads + u.head * G + row;
      p.out[orow * D + d] = __builtin_bit_cast(uint16_t, (__bf16)val);
      if (p.lse != nullptr && d == 0) p.lse[orow] = lse_v;
    } else {
      p.o_part[((size_t)u.part * kRows + row) * D + d] = val;
      if (d == 0) p.lse_part[(size_t)u.part * kRows + row] = lse_v;
    }
  }
}

// ---------------------------------------------------------------- bf16 pool

// Registers of one page pair as loaded.
template <int D>
struct PairRegs {
  uint4 ka[D / 32], kb[D / 32];  // K A-operands of the two pages, one per 32-dim step
  uint2 va[D / 16], vb[D / 16];  // V^T: slots 4g..4g+3 of each page, one per 16-dim block
};

struct PlainLoads {
  __device__ bool operator()() const { return false; }
};

// One unit on NW waves; wave w takes page pairs w, w + NW, ...  nt: asked once the first
// (plain) loads are on their way, whether to read the further pages non-temporally; uniform.
template <int D, int NW, bool NANS, class Nt>
__device__ __forceinline__ void decode_unit(const DecodeArgs& p, const DecodeUnit& u, CombineShared<D, NW> sm, Nt&& nt) {
  constexpr int QS = D / 32;   // QK reduction steps
  constexpr int DB = D / 16;   // PV output blocks
  constexpr int PAGE_ELEMS = kPageSize * D;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n = lane & 15;   // A row (key within a page) / B, C column (query row)
  const int g = lane >> 4;   // lane group
  const int G = p.group;

  // Q^T B-operands: dims 32 s + 8 g .. +8 of query row n (zero past the group)
  bf16x8 qf[QS];
  {
    const bool valid = n < G;
    const uint4* src = (const uint4*)(p.q + ((size_t)u.qo_row * p.num_q_heads + u.head * G + (valid ? n : 0)) * D + 8 * g);
#pragma unroll
    for (int s = 0; s < QS; s++) qf[s] = __builtin_bit_cast(bf16x8, valid ? src[4 * s] : make_uint4(0, 0, 0, 0));
  }

  const size_t head_off = (size_t)u.head * PAGE_ELEMS;
  const size_t page_stride = (size_t)p.num_kv_heads * PAGE_ELEMS;
  const const_i32_ptr pages = (const_i32_ptr)p.page_ids + u.page_base;
  const int last_page = (u.key_end - 1) / kPageSize;
  const int lp0 = u.key_begin / kPageSize;
  const int n_pairs = (u.key_end - u.key_begin + 2 * kPageSize - 1) / (2 * kPageSize);

  // element offsets of the (page, KV head) blocks of pair `pair`; pages past the
  // end repeat the last one (their keys are masked)
  auto blocks = [&](int pair, size_t& pa, size_t& pb) {
    int la = lp0 + 2 * pair, lb = la + 1;
    la = la < last_page ? la : last_page;
    lb = lb < last_page ? lb : last_page;
    pa = (size_t)(uint32_t)pages[la] * page_stride + head_off;
    pb = (size_t)(uint32_t)pages[lb] * page_stride + head_off;
  };
  auto load_k = [&](size_t pa, size_t pb, PairRegs<D>& r, auto nt_flag) {
    constexpr bool NT = decltype(nt_flag)::value;
    const uint16_t* k = (const uint16_t*)p.k_pool;
#pragma unroll
    for (int s = 0; s < QS; s++) {
      r.ka[s] = load16<NT>(k + pa + n * D + 32 * s + 8 * g);
      r.kb[s] = load16<NT>(k + pb + n * D + 32 * s + 8 * g);
    }
  };
  auto load_v = [&](size_t pa, size_t pb, PairRegs<D>& r, auto nt_flag) {
    constexpr bool NT = decltype(nt_flag)::value;
    const uint16_t* v = (const uint16_t*)p.v_pool;
#pragma unroll
    for (int b = 0; b < DB; b++) {
      r.va[b] = load8<NT>(v + pa + (16 * b + n) * kPageSize + 4 * g);
      r.vb[b] = load8<NT>(v + pb + (16 * b + n) * kPageSize + 4 * g);
    }
  };

  f32x4 o[DB];
#pragma unroll
  for (int b = 0; b < DB; b++) o[b] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m_run = -INFINITY, l_run = 0.f;
  const float scale = p.scale_log2;

  // Pair `pair` from r; the registers are refilled with pair `next` (if < n_pairs)
  // as soon as the products have read them, so the loads of the next pair are in
  // flight for the rest of this one.
  auto compute = [&](int pair, int next, PairRegs<D>& r, auto nt_flag) {
    size_t na = 0, nb = 0;
    const bool more = next < n_pairs;  // uniform
    if (more) blocks(next, na, nb);
    f32x4 sa = {0.f, 0.f, 0.f, 0.f}, sb = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < QS; s++) {
      sa = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, r.ka[s]), qf[s], sa, 0, 0, 0);
      sb = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, r.kb[s]), qf[s], sb, 0, 0, 0);
    }
    if (more) load_k(na, nb, r, nt_flag);
    uint2 va[DB], vb[DB];
#pragma unroll
    for (int b = 0; b < DB; b++) {
      va[b] = r.va[b];
      vb[b] = r.vb[b];
    }
    if (more) load_v(na, nb, r, nt_flag);
    // keys of this lane: 4g + i of page a (key0) and of page b (key0 + 16)
    const int key0 = u.key_begin + 32 * pair + 4 * g;
    const bool tail = u.key_begin + 32 * (pair + 1) > u.key_end;  // uniform
    if (tail) {
#pragma unroll
      for (int i = 0; i < 4; i++) {
        if (key0 + i >= u.key_end) sa[i] = -INFINITY;
        if (key0 + 16 + i >= u.key_end) sb[i] = -INFINITY;
      }
      // zero V of keys past the end: unwritten slots may hold NaN
      const uint32_t ma0 = (key0 + 0 < u.key_end ? 0xFFFFu : 0u) | (key0 + 1 < u.key_end ? 0xFFFF0000u : 0u);
      const uint32_t ma1 = (key0 + 2 < u.key_end ? 0xFFFFu : 0u) | (key0 + 3 < u.key_end ? 0xFFFF0000u : 0u);
      const uint32_t mb0 = (key0 + 16 < u.key_end ? 0xFFFFu : 0u) | (key0 + 17 < u.key_end ? 0xFFFF0000u : 0u);
      const uint32_t mb1 = (key0 + 18 < u.key_end ? 0xFFFFu : 0u) | (key0 + 19 < u.key_end ? 0xFFFF0000u : 0u);
#pragma unroll
      for (int b = 0; b < DB; b++) {
        va[b].x &= ma0;
        va[b].y &= ma1;
        vb[b].x &= mb0;
        vb[b].y &= mb1;
      }
    }
    float mx = fmaxf(fmaxf(fmaxf(sa[0], sa[1]), fmaxf(sa[2], sa[3])), fmaxf(fmaxf(sb[0], sb[1]), fmaxf(sb[2], sb[3])));
    mx = group_max(mx) * scale;
    if (__any(mx > m_run)) {
      const float m_new = fmaxf(m_run, mx);
      // 0 when m_run = -inf; a NaN when both are, for a row without a score above -inf
      const float alpha = NANS && m_new == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m_run - m_new);
      l_run *= alpha;
#pragma unroll
      for (int b = 0; b < DB; b++) o[b] *= alpha;
      m_run = m_new;
    }
    // a row whose keys so far are all masked keeps m_run = -inf: its p are 0
    const float neg = m_run == -INFINITY ? 0.f : -m_run;
    float pa[4], pb[4];
#pragma unroll
    for (int i = 0; i < 4; i++) {
      pa[i] = __builtin_amdgcn_exp2f(__builtin_fmaf(sa[i], scale, neg));
      pb[i] = __builtin_amdgcn_exp2f(__builtin_fmaf(sb[i], scale, neg));
    }
    const uint4 pw = make_uint4(pack2(pa[0], pa[1]), pack2(pa[2], pa[3]), pack2(pb[0], pb[1]), pack2(pb[2], pb[3]));
    const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
    l_run = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pw.x), ones, l_run, false);
    l_run = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pw.y), ones, l_run, false);
    l_run = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pw.z), ones, l_run, false);
    l_run = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pw.w), ones, l_run, false);
    const bf16x8 pbv = __builtin_bit_cast(bf16x8, pw);
#pragma unroll
    for (int b = 0; b < DB; b++) {
      const uint4 vv = make_uint4(va[b].x, va[b].y, vb[b].x, vb[b].y);
      o[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, vv), pbv, o[b], 0, 0, 0);
    }
  };

  PairRegs<D> r;
  if (wave < n_pairs) {
    size_t pa, pb;
    blocks(wave, pa, pb);
    load_k(pa, pb, r, std::false_type{});
    load_v(pa, pb, r, std::false_type{});
  }
  if (nt())
    for (int j = wave; j < n_pairs; j += NW) compute(j, j + NW, r, std::true_type{});
  else
    for (int j = wave; j < n_pairs; j += NW) compute(j, j + NW, r, std::false_type{});

  combine_waves<D, NW, NANS>(p, u, sm, o, m_run, l_run, 1.0f, 0.f);
}

// ---------------------------------------------------------------- fp8 pool
//
// A wave takes 64 keys (four pages) a step, so that every load is 16 bytes per lane
// and a step has as many bytes in flight as a bf16 pair:
//   * K: MFMA j of a k-step holds slots 4j .. 4j+3 of each of the four pages: A row m
//     is slot 4j + m % 4 of page m / 4.  A lane's 16 codes (dims 64 i + 16 g .. +15 of
//     its row) feed two k-steps; Q's dims are loaded in the same order.
//   * In the S^T result lane group g then holds page g: S_j[i] is slot 4j + i.  Its P
//     values of S_0, S_1 (slots 0..7) and S_2, S_3 (slots 8..15) are the B operands of two
//     PV products, whose A operands are the two halves of one 16-code load of V^T
//     (dim 16 b + n of page g).
// The codes are converted exactly (every e4m3 value is a bf16 value); k_scale goes
// into the softmax scale, v_scale into the result.
// HBM bound.  24 agents with 16k-131k contexts, 64/8/128 heads, 3.14 GB: 722 us with
// 8-byte K and 4-byte V loads of 32 keys a step, 542 us (5.8 TB/s) now.  Four workgroups
// per CU instead of two spill and take 864 us.
template <int D>
struct QuadRegs {
  uint4 k[4][D / 64];  // K codes: MFMA j, 64-dim step i
  uint4 v[D / 16];     // V^T codes: all 16 slots of the lane's dim of page g
};

template <int D, int NW, bool NANS, class Nt>
__device__ __forceinline__ void decode_unit_fp8(const DecodeArgs& p, const DecodeUnit& u, CombineShared<D, NW> sm,
                                                Nt&& nt) {
  constexpr int KS = D / 64;  // K loads per MFMA row block
  constexpr int DB = D / 16;  // PV output blocks
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n = lane & 15;  // A row / B, C column (query row)
  const int g = lane >> 4;  // lane group
  const int G = p.group;

  // Q^T B-operands: k-step (i, h) takes dims 64 i + 16 g + 8 h .. +8 of query row n
  bf16x8 qf[KS][2];
  {
    const bool valid = n < G;
    const uint4* src =
        (const uint4*)(p.q + ((size_t)u.qo_row * p.num_q_heads + u.head * G + (valid ? n : 0)) * D + 16 * g);
#pragma unroll
    for (int i = 0; i < KS; i++)
#pragma unroll
      for (int h = 0; h < 2; h++)
        qf[i][h] = __builtin_bit_cast(bf16x8, valid ? src[8 * i + h] : make_uint4(0, 0, 0, 0));
  }

  const uint32_t page_bytes = (uint32_t)p.num_kv_heads * (kPageSize * D);
  const const_i32_ptr pages = (const_i32_ptr)p.page_ids + u.page_base;
  const int last_page = (u.key_end - 1) / kPageSize;
  const int lp0 = u.key_begin / kPageSize;
  const int n_quads = (u.key_end - u.key_begin + 4 * kPageSize - 1) / (4 * kPageSize);
  // the lane's K row and V dim inside a (page, KV head) block
  const char* kbase = (const char*)p.k_pool + (size_t)u.head * (kPageSize * D) + (n & 3) * D + 16 * g;
  const char* vbase = (const char*)p.v_pool + (size_t)u.head * (kPageSize * D) + n * kPageSize;

  // page ids of quad `quad` (pages past the end repeat the last one, their keys are
  // masked), and from them the lane's K page (n / 4) and V page (g)
  typedef uint32_t ids_t __attribute__((ext_vector_type(4)));
  auto ids_of = [&](int quad) {
    const int l = lp0 + 4 * quad;
    auto at = [&](int i) { return (uint32_t)pages[l + i < last_page ? l + i : last_page]; };
    return ids_t{at(0), at(1), at(2), at(3)};
  };
  auto pick = [](const ids_t& w, bool odd, bool high) {
    const uint32_t lo = odd ? w.y : w.x, hi = odd ? w.w : w.z;
    return high ? hi : lo;
  };
  const bool k_odd = n & 4, k_high = n & 8, v_odd = g & 1, v_high = g & 2;
  auto load_k = [&](const ids_t& w, QuadRegs<D>& r, auto nt_flag) {
    constexpr bool NT = decltype(nt_flag)::value;
    const char* src = kbase + (uint64_t)pick(w, k_odd, k_high) * page_bytes;
#pragma unroll
    for (int j = 0; j < 4; j++)
#pragma unroll
      for (int i = 0; i < KS; i++) r.k[j][i] = load16<NT>(src + 4 * j * D + 64 * i);
  };
  auto load_v = [&](const ids_t& w, QuadRegs<D>& r, auto nt_flag) {
    constexpr bool NT = decltype(nt_flag)::value;
    const char* src = vbase + (uint64_t)pick(w, v_odd, v_high) * page_bytes;
#pragma unroll
    for (int b = 0; b < DB; b++) r.v[b] = load16<NT>(src + 256 * b);
  };

  f32x4 o[DB];
#pragma unroll
  for (int b = 0; b < DB; b++) o[b] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m_run = -INFINITY, l_run = 0.f;
  const float scale = p.scale_log2 * p.k_scale[u.head];

  // Quad `quad` from r; its registers are refilled with quad `next` (if < n_quads) as
  // soon as the products have read them.  TAIL: the quad reaches past key_end.  (A template
  // flag and not a branch: masked under a branch in the loop, the results are the same bits,
  // but 8 registers more go over it: 100 agents on 8/2/64 heads 146 us, 135 so.)
  auto compute = [&](int quad, int next, QuadRegs<D>& r, auto tail_flag, auto nt_flag) {
    constexpr bool TAIL = decltype(tail_flag)::value;
    const bool more = next < n_quads;  // uniform
    ids_t nx{};
    if (more) nx = ids_of(next);
    f32x4 s[4];
#pragma unroll
    for (int j = 0; j < 4; j++) {
      s[j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int i = 0; i < KS; i++) {
        const uint4 c = r.k[j][i];
        s[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, fp8x8_bf16(make_uint2(c.x, c.y))),
                                                       qf[i][0], s[j], 0, 0, 0);
        s[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, fp8x8_bf16(make_uint2(c.z, c.w))),
                                                       qf[i][1], s[j], 0, 0, 0);
      }
    }
    if (more) load_k(nx, r, nt_flag);
    const int key0 = u.key_begin + 64 * quad + 16 * g;  // slot 0 of the lane group's page
    if constexpr (TAIL) {
#pragma unroll
      for (int j = 0; j < 4; j++)
#pragma unroll
        for (int i = 0; i < 4; i++)
          if (key0 + 4 * j + i >= u.key_end) s[j][i] = -INFINITY;
    }
    float mx = -INFINITY;
#pragma unroll
    for (int j = 0; j < 4; j++)
#pragma unroll
      for (int i = 0; i < 4; i++) mx = fmaxf(mx, s[j][i]);
    mx = group_max(mx) * scale;
    if (__any(mx > m_run)) {
      const float m_new = fmaxf(m_run, mx);
      // 0 when m_run = -inf; a NaN when both are, for a row without a score above -inf
      const float alpha = NANS && m_new == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m_run - m_new);
      l_run *= alpha;
#pragma unroll
      for (int b = 0; b < DB; b++) o[b] *= alpha;
      m_run = m_new;
    }
    const float neg = m_run == -INFINITY ? 0.f : -m_run;
    const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
    uint32_t pw[8];  // P of slots 2 e, 2 e + 1
#pragma unroll
    for (int e = 0; e < 8; e++) {
      const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[e / 2][2 * (e % 2)], scale, neg));
      const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[e / 2][2 * (e % 2) + 1], scale, neg));
      pw[e] = pack2(p0, p1);
      l_run = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pw[e]), ones, l_run, false);
    }
    const bf16x8 pa = __builtin_bit_cast(bf16x8, make_uint4(pw[0], pw[1], pw[2], pw[3]));
    const bf16x8 pb = __builtin_bit_cast(bf16x8, make_uint4(pw[4], pw[5], pw[6], pw[7]));
    uint32_t mask[4];  // zeroes V of keys past the end: unwritten slots may hold NaN codes
    if constexpr (TAIL) {
#pragma unroll
      for (int e = 0; e < 4; e++) {
        const int left = u.key_end - key0 - 4 * e;  // live slots of this dword
        mask[e] = left >= 4 ? 0xFFFFFFFFu : left <= 0 ? 0u : (1u << (8 * left)) - 1u;
      }
    }
#pragma unroll
    for (int b = 0; b < DB; b++) {
      uint4 c = r.v[b];
      if constexpr (TAIL) c = make_uint4(c.x & mask[0], c.y & mask[1], c.z & mask[2], c.w & mask[3]);
      o[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, fp8x8_bf16(make_uint2(c.x, c.y))), pa,
                                                     o[b], 0, 0, 0);
      o[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, fp8x8_bf16(make_uint2(c.z, c.w))), pb,
                                                     o[b], 0, 0, 0);
    }
    if (more) load_v(nx, r, nt_flag);
  };

  QuadRegs<D> r;
  if (wave < n_quads) {
    const ids_t w = ids_of(wave);
    load_k(w, r, std::false_type{});
    load_v(w, r, std::false_type{});
  }
  const int n_full = (u.key_end - u.key_begin) / (4 * kPageSize);  // at most the last quad is not full
  int j = wave;
  if (nt())
    for (; j < n_full; j += NW) compute(j, j + NW, r, std::false_type{}, std::true_type{});
  else
    for (; j < n_full; j += NW) compute(j, j + NW, r, std::false_type{}, std::false_type{});
  if (j < n_quads) compute(j, j + NW, r, std::true_type{}, std::false_type{});
  combine_waves<D, NW, NANS>(p, u, sm, o, m_run, l_run, p.v_scale[u.head], __builtin_nanf(""));
}


}  // namespace decode
}  // namespace
}  // namespace kvx
