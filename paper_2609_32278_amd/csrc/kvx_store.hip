// KV store into the paged pool and raw page I/O, gfx950 (CDNA4).
//
// Prefill materialises the suffix's K/V in every attention layer (paper,
// Section 2); store_kv writes them into the request's pages so that the next
// attention pass -- and every later turn that reuses this prefix -- reads them
// from the pool.  HBM-bound: each element is read once and written once.
//
// Pool layout: K [page][kv_head][slot][dim], V [page][kv_head][dim][slot].
// One workgroup handles one page of one request for one group of 4 KV heads
// (head_dim 128) or 8 (head_dim 64) -- grid x = the page, y = the head group, so
// that a batch touching few pages still fills the chip -- and issues all of its
// loads before using any (four K and four V 16-byte loads in flight per thread; its
// 16-byte stores, like the fused store's, are non-temporal: 48k tokens of 8/1/128 heads
// 58 -> 46 us, 27k tokens of 64/8/128 heads 221 -> 216 us, 16k tokens of 8 K/V heads 24.6
// -> 21.0 us, and no turn whose attention reads them back got slower):
// K rows are copied with 16-byte accesses, V rows are staged in LDS and written
// out transposed, one 16-slot column (32 bytes bf16 / 16 bytes fp8) per dim.
// fp8 pool: code = e4m3_rne(clamp(x * inv_scale_h, -448, 448)) with the
// hardware converter v_cvt_pk_fp8_f32 (OCP e4m3 on gfx950).

#include <type_traits>

#include "kvx_internal.h"

namespace kvx {
namespace {

constexpr int kStoreThreads = 256;

// 16-byte accesses; NT: non-temporal, for data that no cache need keep.
template <bool NT>
__device__ __forceinline__ uint4 load16(const void* p) {
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  if constexpr (NT) return __builtin_bit_cast(uint4, __builtin_nontemporal_load((const u32x4*)p));
  else return *(const uint4*)p;
}
template <bool NT>
__device__ __forceinline__ void store16(void* p, uint4 x) {
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  if constexpr (NT) __builtin_nontemporal_store(__builtin_bit_cast(u32x4, x), (u32x4*)p);
  else *(uint4*)p = x;
}

__device__ __forceinline__ float bf16_to_f32(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

__device__ __forceinline__ float clamp448(float x) { return fminf(fmaxf(x, -448.0f), 448.0f); }

// 4 floats -> 4 e4m3 codes (byte i = value i)
__device__ __forceinline__ uint32_t e4m3x4(float a, float b, float c, float d) {
  int r = __builtin_amdgcn_cvt_pk_fp8_f32(clamp448(a), clamp448(b), 0, false);
  r = __builtin_amdgcn_cvt_pk_fp8_f32(clamp448(c), clamp448(d), r, true);
  return (uint32_t)r;
}

// Write the staged V rows vs[slot][dim] of one (page, head) block as the pool's
// [dim][slot] columns, 8 slots per thread and step (16 bytes bf16 / 8 bytes fp8);
// only slots in [slot_begin, slot_end) are written.
template <int D, bool FP8>
__device__ __forceinline__ void write_vt(const uint16_t (&vs)[kPageSize][D + 8], void* v_pool, size_t blk,
                                         int slot_begin, int slot_end, float vinv) {
  const bool full = slot_begin == 0 && slot_end == kPageSize;
  for (int c = threadIdx.x; c < 2 * D; c += kStoreThreads) {
    const int d = c / 2, half = c % 2;
    const int s0 = half * 8;
    if (s0 + 8 <= slot_begin || s0 >= slot_end) continue;
    float x[8];
    uint16_t raw[8];
#pragma unroll
    for (int e = 0; e < 8; e++) {
      raw[e] = vs[s0 + e][d];
      x[e] = bf16_to_f32(raw[e]) * vinv;
    }
    const bool whole = full || (s0 >= slot_begin && s0 + 8 <= slot_end);
    if constexpr (FP8) {
      uint8_t* dst = (uint8_t*)v_pool + blk + (size_t)d * kPageSize + s0;
      uint2 code;
      code.x = e4m3x4(x[0], x[1], x[2], x[3]);
      code.y = e4m3x4(x[4], x[5], x[6], x[7]);
      if (whole) {
        *(uint2*)dst = code;
      } else {
        const uint8_t* cb = (const uint8_t*)&code;
        for (int e = 0; e < 8; e++)
          if (s0 + e >= slot_begin && s0 + e < slot_end) dst[e] = cb[e];
      }
    } else {
      uint16_t* dst = (uint16_t*)v_pool + blk + (size_t)d * kPageSize + s0;
      if (whole) {
        uint4 w;
        w.x = raw[0] | ((uint32_t)raw[1] << 16);
        w.y = raw[2] | ((uint32_t)raw[3] << 16);
        w.z = raw[4] | ((uint32_t)raw[5] << 16);
        w.w = raw[6] | ((uint32_t)raw[7] << 16);
        store16<true>(dst, w);
      } else {
        for (int e = 0; e < 8; e++)
          if (s0 + e >= slot_begin && s0 + e < slot_end) dst[e] = raw[e];
      }
    }
  }
}

// The unit of workgroup b of a small batch (see StoreReqs); uniform.
__device__ __forceinline__ RopeUnit inline_unit(const StoreReqs& rq, int b) {
  int lo = 0, hi = rq.n;  // request r with first[r] <= b < first[r + 1]
  while (hi - lo > 1) {
    const int mid = (lo + hi) / 2;
    if (rq.first[mid] <= b) lo = mid;
    else hi = mid;
  }
  const int P = rq.prefix[lo], L = rq.end[lo];
  const int lp = P / kPageSize + (b - rq.first[lo]);
  RopeUnit u;
  u.pos_slot0 = lp * kPageSize;
  u.row_slot0 = rq.qo[lo] + u.pos_slot0 - P;
  u.page_pos = rq.page_base[lo] + lp;
  u.slot_begin = (P > u.pos_slot0 ? P : u.pos_slot0) - u.pos_slot0;
  u.slot_end = (L < u.pos_slot0 + kPageSize ? L : u.pos_slot0 + kPageSize) - u.pos_slot0;
  return u;
}

template <int D, bool FP8>
__global__ __launch_bounds__(kStoreThreads) void store_kv_kernel(StoreParams p) {
  constexpr int CPR = D / 8;                          // 16-byte chunks per bf16 row
  constexpr int CHUNKS = kPageSize * CPR;             // per head
  constexpr int HB = 4 * kStoreThreads / CHUNKS;      // heads per pass: 4 (D = 128), 8 (D = 64)
  constexpr int PER = HB * CHUNKS / kStoreThreads;    // chunks per thread and pass
  static_assert(PER == 4, "four K and four V loads in flight per thread");
  // V rows of this page for the pass's heads, staged for the transpose: [head][16 slots][D] bf16
  __shared__ __attribute__((aligned(16))) uint16_t vs[HB][kPageSize][D + 8];
  StoreUnit su;
  if (p.reqs.n > 0) {
    const RopeUnit u = inline_unit(p.reqs, blockIdx.x);
    su = StoreUnit{u.row_slot0, u.page_pos, u.slot_begin, u.slot_end};
  } else {
    su = p.units[blockIdx.x];
  }
  const int page = p.page_ids[su.page_pos];
  const int H = p.num_kv_heads;

  {
    const int h0 = blockIdx.y * HB;
    // every load of the pass is issued before any of them is used
    uint4 kx[PER], vx[PER];
#pragma unroll
    for (int j = 0; j < PER; j++) {
      const int i = threadIdx.x + j * kStoreThreads;
      const int hd = h0 + i / CHUNKS, slot = (i % CHUNKS) / CPR, cc = i % CPR;
      kx[j] = vx[j] = make_uint4(0, 0, 0, 0);
      if (hd < H && slot >= su.slot_begin && slot < su.slot_end) {
        const size_t src = ((size_t)(su.row_slot0 + slot) * H + hd) * D + cc * 8;
        kx[j] = *(const uint4*)(p.k_ext + src);
        vx[j] = *(const uint4*)(p.v_ext + src);
      }
    }
#pragma unroll
    for (int j = 0; j < PER; j++) {
      const int i = threadIdx.x + j * kStoreThreads;
      const int hb = i / CHUNKS, hd = h0 + hb, slot = (i % CHUNKS) / CPR, cc = i % CPR;
      if (hd >= H) continue;
      if (slot >= su.slot_begin && slot < su.slot_end) {
        const size_t blk = ((size_t)page * H + hd) * (size_t)(kPageSize * D);
        if constexpr (FP8) {
          const float kinv = p.k_inv_scale[hd];
          const uint16_t* ke = (const uint16_t*)&kx[j];
          uint2 code;
          code.x = e4m3x4(bf16_to_f32(ke[0]) * kinv, bf16_to_f32(ke[1]) * kinv,
                          bf16_to_f32(ke[2]) * kinv, bf16_to_f32(ke[3]) * kinv);
          code.y = e4m3x4(bf16_to_f32(ke[4]) * kinv, bf16_to_f32(ke[5]) * kinv,
                          bf16_to_f32(ke[6]) * kinv, bf16_to_f32(ke[7]) * kinv);
          *(uint2*)((uint8_t*)p.k_pool + blk + (size_t)slot * D + cc * 8) = code;
        } else {
          store16<true>((uint16_t*)p.k_pool + blk + (size_t)slot * D + cc * 8, kx[j]);
        }
      }
      *(uint4*)(&vs[hb][slot][cc * 8]) = vx[j];
    }
    __syncthreads();
    for (int hb = 0; hb < HB && h0 + hb < H; hb++) {
      const int hd = h0 + hb;
      const size_t blk = ((size_t)page * H + hd) * (size_t)(kPageSize * D);
      write_vt<D, FP8>(vs[hb], p.v_pool, blk, su.slot_begin, su.slot_end, FP8 ? p.v_inv_scale[hd] : 1.0f);
    }
  }
}

// ---------------------------------------------------------------- fused RoPE store
//
// The step before attention, fused into the store (the models the paper serves
// normalise and rotate Q and K before K is cached; the paper itself describes
// neither step): every Q and K head row of the unit's tokens is optionally
// RMS-normalised, rotated by its absolute position, and then written -- Q to
// q_out as bf16, K into the pool as store_kv would store it.  V is stored as by
// store_kv.  Arithmetic is fp32; each angle is reduced to [-pi, pi] in fp64 from
// the plane's rate in revolutions per position, so positions far past 2^24
// keep full precision.  Results are rounded once (RNE bf16 or e4m3).
//
// Work split: one workgroup per touched page and group of heads (Q groups, K groups,
// V groups).  One workgroup per page walking all heads left a batch of a few dozen
// to a few hundred pages with one long serial chain per CU -- a V head after another,
// two barriers each (1.0 TB/s at 150 pages, 49 MB); a group per workgroup runs the same
// batch at 3.0 TB/s (42.6 -> 16.4 us) and 1700 pages of 64+8 heads at 4.8 TB/s (249 -> 237 us,
// where a 4 GiB copy reaches 4.8 TB/s).  The price is that each group forms the page's
// angles again, which its first loads overlap.
//
// A head row of D bf16 values is D/8 16-byte chunks held by D/8 consecutive
// lanes; the RMS sum is reduced across those lanes, and in the half layout a
// chunk of the first half meets its plane partners in the chunk rotary_dim/16
// lanes further on (one lane shuffle per value).

constexpr int kRopeBatch = 4;  // chunks per thread in flight
constexpr int kRopeVHeads = 4;   // V heads per workgroup

template <int D, bool INTERLEAVED>
struct RopeLane {
  static constexpr int CPR = D / 8;
  int cc;           // chunk of the row this lane handles (fixed for the thread)
  int partner;      // lane holding the plane partners (half layout)
  int jb;           // first plane of the chunk
  bool rot;         // the chunk lies inside rotary_dim
  float sgn;        // half layout: -1 for the plane's first dims, +1 for its second

  __device__ RopeLane(int rotary_dim) {
    cc = threadIdx.x % CPR;
    const int lane = threadIdx.x & 63;
    if constexpr (INTERLEAVED) {
      rot = cc < (rotary_dim >> 3);
      jb = 4 * cc;
      partner = lane;
      sgn = 0.0f;
    } else {
      const int r16 = rotary_dim >> 4;
      const bool first = cc < r16;
      rot = cc < 2 * r16;
      jb = first ? 8 * cc : 8 * (cc - r16);
      partner = lane + (first ? r16 : (rot ? -r16 : 0));
      sgn = first ? -1.0f : 1.0f;
    }
  }
};

// x: the 8 values of this lane's chunk of one row at `slot`; in place -> rotated.
// Every lane of the row must execute this (shuffles).
template <int D, bool INTERLEAVED>
__device__ __forceinline__ void rope_chunk(float (&x)[8], const RopeLane<D, INTERLEAVED>& rl,
                                           const float2* cs_slot) {
  if constexpr (INTERLEAVED) {
#pragma unroll
    for (int i = 0; i < 4; i++) {
      const float2 t = rl.rot ? cs_slot[rl.jb + i] : make_float2(1.0f, 0.0f);
      const float a = x[2 * i], b = x[2 * i + 1];
      x[2 * i] = a * t.x - b * t.y;
      x[2 * i + 1] = a * t.y + b * t.x;
    }
  } else {
    float pe[8];
#pragma unroll
    for (int e = 0; e < 8; e++) pe[e] = __shfl(x[e], rl.partner, 64);
#pragma unroll
    for (int e = 0; e < 8; e++) {
      const float2 t = rl.rot ? cs_slot[rl.jb + e] : make_float2(1.0f, 0.0f);
      // first dims: a cos - b sin (b = partner); second dims: b cos + a sin (a = partner)
      x[e] = x[e] * t.x + rl.sgn * (pe[e] * t.y);
    }
  }
}

// Normalise and rotate `nh` heads from h0 on (nh <= 1 << lg) of the unit's ntok tokens
// (src: the first token's row, [token][heads][D] bf16) and hand each chunk's results
// to out(token, head, chunk, y).  The first loads are issued before angles() -- which
// fills cs and ends in a barrier -- so that they are in flight meanwhile.
template <int D, bool INTERLEAVED, class Angles, class Out>
__device__ __forceinline__ void rope_rows(const uint16_t* __restrict__ src, int ntok, int heads, int h0, int nh, int lg,
                                          int slot_begin, const float2 (*cs)[kRopeMaxPlanes],
                                          const uint16_t* norm_w, float eps, int rotary_dim, Angles&& angles,
                                          Out&& out) {
  constexpr int CPR = D / 8;
  const RopeLane<D, INTERLEAVED> rl(rotary_dim);
  // row index rr = token << lg | head of the group; rows past the group's heads idle
  const int n = ntok << lg;
  constexpr int ROWS = kStoreThreads / CPR;  // rows per step
  const int r0 = threadIdx.x / CPR;
  auto load = [&](int rr) {
    const int tok = rr >> lg, hh = rr & ((1 << lg) - 1);
    return rr < n && hh < nh ? *(const uint4*)(src + ((size_t)tok * heads + h0 + hh) * D + rl.cc * 8)
                             : make_uint4(0, 0, 0, 0);
  };
  uint4 raw[kRopeBatch];
#pragma unroll
  for (int b = 0; b < kRopeBatch; b++) raw[b] = load(r0 + b * ROWS);
  float w[8];
  if (norm_w) {
    const uint4 wr = *(const uint4*)(norm_w + rl.cc * 8);
    const uint16_t* wh = (const uint16_t*)&wr;
#pragma unroll
    for (int e = 0; e < 8; e++) w[e] = bf16_to_f32(wh[e]);
  }
  angles();
  for (int c0 = r0; c0 - r0 < n; c0 += kRopeBatch * ROWS) {
    uint4 next[kRopeBatch];
#pragma unroll
    for (int b = 0; b < kRopeBatch; b++) next[b] = load(c0 + (kRopeBatch + b) * ROWS);
#pragma unroll
    for (int b = 0; b < kRopeBatch; b++) {
      const int rr = c0 + b * ROWS;
      if (rr - r0 >= n) break;  // uniform
      const int tok = rr >> lg, hh = rr & ((1 << lg) - 1);
      const uint16_t* h16 = (const uint16_t*)&raw[b];
      float x[8];
#pragma unroll
      for (int e = 0; e < 8; e++) x[e] = bf16_to_f32(h16[e]);
      if (norm_w) {
        float ss = 0.0f;
#pragma unroll
        for (int e = 0; e < 8; e++) ss = fmaf(x[e], x[e], ss);
#pragma unroll
        for (int m = 1; m < CPR; m <<= 1) ss += __shfl_xor(ss, m, 64);
        const float inv = 1.0f / sqrtf(ss * (1.0f / D) + eps);
#pragma unroll
        for (int e = 0; e < 8; e++) x[e] = (x[e] * inv) * w[e];
      }
      rope_chunk<D, INTERLEAVED>(x, rl, cs[slot_begin + (rr < n ? tok : 0)]);
      if (rr < n && hh < nh) out(tok, h0 + hh, rl.cc, x);
    }
#pragma unroll
    for (int b = 0; b < kRopeBatch; b++) raw[b] = next[b];
  }
}

__device__ __forceinline__ uint4 pack_bf16x8(const float (&y)[8]) {
  uint4 r;
  uint32_t* w = (uint32_t*)&r;
#pragma unroll
  for (int i = 0; i < 4; i++) {
    const __bf16 lo = (__bf16)y[2 * i], hi = (__bf16)y[2 * i + 1];
    w[i] = (uint32_t)__builtin_bit_cast(uint16_t, lo) | ((uint32_t)__builtin_bit_cast(uint16_t, hi) << 16);
  }
  return r;
}

// Grid: x = the unit (a touched page), y = a group of heads: first the groups of
// 1 << p.lg_q Q heads, then those of 1 << p.lg_k K heads, then those of HB V heads.  With
// p.whole_page, y = 0 takes them all, one after another, with the angles formed once.
template <int D, bool FP8, bool INTERLEAVED>
__global__ __launch_bounds__(kStoreThreads) void store_kv_rope_kernel(RopeParams p) {
  constexpr int CPR = D / 8;
  constexpr int HB = kRopeVHeads;
  constexpr int VCHUNKS = kPageSize * CPR;  // 16-byte chunks of one head's V rows
  constexpr int PER = HB * VCHUNKS / kStoreThreads;
  union Shared {
    float2 cs[kPageSize][kRopeMaxPlanes];  // (cos, sin) of every live slot and plane
    uint16_t vs[HB][kPageSize][D + 8];     // V rows staged for the transpose
  };
  __shared__ __attribute__((aligned(16))) Shared sm;
  const RopeUnit u = p.reqs.n > 0 ? inline_unit(p.reqs, blockIdx.x) : p.units[blockIdx.x];
  const int ntok = u.slot_end - u.slot_begin;
  const int Hq = p.num_q_heads, H = p.num_kv_heads;
  const int row0 = u.row_slot0 + u.slot_begin;  // first suffix row of the unit
  const int nq = (Hq + (1 << p.lg_q) - 1) >> p.lg_q, nk = (H + (1 << p.lg_k) - 1) >> p.lg_k;
  const int y = blockIdx.y;
  const bool whole = p.whole_page != 0;
  bool have_angles = false;

  auto angles = [&]() {
    if (have_angles) return;  // uniform
    have_angles = true;
    const int planes = p.rotary_dim / 2;
    for (int e = threadIdx.x; e < ntok * planes; e += kStoreThreads) {
      const int s = u.slot_begin + e / planes, j = e % planes;
      double rev = (double)(u.pos_slot0 + s) * p.rev_freq[j];  // exact position times the rate
      rev -= rint(rev);                                          // [-1/2, 1/2] turn, exact
      float sn, cn;
      sincospif(2.0f * (float)rev, &sn, &cn);
      sm.cs[s][j] = make_float2(cn, sn);
    }
    __syncthreads();
  };

  if (y < nq || (whole && Hq > 0)) {
    const int hpg = 1 << p.lg_q, h0 = whole ? 0 : y << p.lg_q, nh = Hq - h0 < hpg ? Hq - h0 : hpg;
    uint16_t* qo = p.q_out + (size_t)row0 * Hq * D;
    rope_rows<D, INTERLEAVED>(p.q + (size_t)row0 * Hq * D, ntok, Hq, h0, nh, p.lg_q, u.slot_begin, sm.cs, p.q_norm,
                              p.norm_eps, p.rotary_dim, angles, [&](int tok, int hd, int cc, const float(&v)[8]) {
                                store16<true>(qo + ((size_t)tok * Hq + hd) * D + cc * 8, pack_bf16x8(v));
                              });
    if (!whole) return;
  }
  const int page = p.page_ids[u.page_pos];
  if (whole || y < nq + nk) {
    const int hpg = 1 << p.lg_k, h0 = whole ? 0 : (y - nq) << p.lg_k, nh = H - h0 < hpg ? H - h0 : hpg;
    rope_rows<D, INTERLEAVED>(
        p.k_ext + (size_t)row0 * H * D, ntok, H, h0, nh, p.lg_k, u.slot_begin, sm.cs, p.k_norm, p.norm_eps,
        p.rotary_dim, angles, [&](int tok, int hd, int cc, const float(&v)[8]) {
          const size_t blk = ((size_t)page * H + hd) * (size_t)(kPageSize * D);
          const int slot = u.slot_begin + tok;
          if constexpr (FP8) {
            const float kinv = p.k_inv_scale[hd];
            uint2 code;
            code.x = e4m3x4(v[0] * kinv, v[1] * kinv, v[2] * kinv, v[3] * kinv);
            code.y = e4m3x4(v[4] * kinv, v[5] * kinv, v[6] * kinv, v[7] * kinv);
            *(uint2*)((uint8_t*)p.k_pool + blk + (size_t)slot * D + cc * 8) = code;
          } else {
            store16<true>((uint16_t*)p.k_pool + blk + (size_t)slot * D + cc * 8, pack_bf16x8(v));
          }
        });
    if (!whole) return;
  }

  // V: HB heads staged in LDS at once and written as [dim][slot] columns
  for (int h0 = whole ? 0 : (y - nq - nk) * HB; h0 < H; h0 += HB) {
    uint4 vx[PER];
#pragma unroll
    for (int j = 0; j < PER; j++) {
      const int i = threadIdx.x + j * kStoreThreads;
      const int hd = h0 + i / VCHUNKS, slot = (i % VCHUNKS) / CPR, cc = i % CPR;
      vx[j] = make_uint4(0, 0, 0, 0);
      if (hd < H && slot >= u.slot_begin && slot < u.slot_end)
        vx[j] = *(const uint4*)(p.v_ext + ((size_t)(u.row_slot0 + slot) * H + hd) * D + cc * 8);
    }
    if (whole) __syncthreads();  // the angles (or the heads before) have been read
#pragma unroll
    for (int j = 0; j < PER; j++) {
      const int i = threadIdx.x + j * kStoreThreads;
      *(uint4*)(&sm.vs[i / VCHUNKS][(i % VCHUNKS) / CPR][(i % CPR) * 8]) = vx[j];
    }
    __syncthreads();
#pragma unroll
    for (int hb = 0; hb < HB; hb++) {
      const int hd = h0 + hb;
      if (hd >= H) break;  // uniform
      const size_t blk = ((size_t)page * H + hd) * (size_t)(kPageSize * D);
      write_vt<D, FP8>(sm.vs[hb], p.v_pool, blk, u.slot_begin, u.slot_end, FP8 ? p.v_inv_scale[hd] : 1.0f);
    }
    if (!whole) return;
  }
}

// Spill / reload of whole pages between the pool and pinned host memory.  One
// workgroup per (page, K|V block): the block is contiguous on both sides, so
// every lane moves 16-byte pieces, four in flight before any store (host memory
// is reached over the host link: latency is long, concurrency hides it).
__global__ __launch_bounds__(256) void page_move_kernel(PageMoveParams p) {
  constexpr int kUnroll = 4;
  const int i = blockIdx.x;
  const int kv = blockIdx.y;  // 0: K block, 1: V block
  const int64_t page = p.page_ids[i];
  uint8_t* dev = (kv == 0 ? p.k_pool : p.v_pool) + page * p.block_bytes;
  uint8_t* host = p.host + ((int64_t)p.slots[i] * 2 + kv) * p.block_bytes;
  const uint8_t* src = p.to_host ? dev : host;
  uint8_t* dst = p.to_host ? host : dev;
  const int64_t pieces = p.block_bytes / 16;
  for (int64_t c0 = threadIdx.x; c0 < pieces; c0 += kUnroll * 256) {
    uint4 x[kUnroll];
#pragma unroll
    for (int u = 0; u < kUnroll; u++) {
      const int64_t c = c0 + u * 256;
      if (c < pieces) x[u] = *(const uint4*)(src + c * 16);
    }
#pragma unroll
    for (int u = 0; u < kUnroll; u++) {
      const int64_t c = c0 + u * 256;
      if (c < pieces) *(uint4*)(dst + c * 16) = x[u];
    }
  }
}

// Raw page copy between canonical [n][Hkv][16][D] buffers and the pool.  INLINE: the ids of
// pages first .. of the buffers are in the arguments.
//
// HBM bound.  A workgroup takes BLOCKS consecutive (page, head) blocks and issues all its loads
// before any store: four 16-byte K and four V pieces per thread.  V is transposed through LDS,
// so that both sides see 16-byte pieces.  The pool's side is non-temporal, which leaves the
// buffers in the Infinity Cache for whoever takes them next.  2000 pages of 8 heads out and
// in again, 524 MB: 141 us one block per workgroup and V an element at a time, 129 us, and
// 97 us (5.4 TB/s) non-temporal.
struct PageIds {
  int32_t first;
  int32_t id[kInlinePages];
};
struct NoPageIds {};
__device__ __forceinline__ int64_t first_page(const PageIds& ids) { return ids.first; }
__device__ __forceinline__ int64_t first_page(const NoPageIds&) { return 0; }
template <int D, int EB, bool INLINE, bool TO_POOL>
__global__ __launch_bounds__(256) void page_io_kernel(PageIoParams p, int32_t n_pages,
                                                      std::conditional_t<INLINE, PageIds, NoPageIds> ids) {
  constexpr int CH = D * EB;            // 16-byte pieces of a block (16 slots x D elements)
  constexpr int PER = 4;                // pieces of K, and of V, per thread
  constexpr int BLOCKS = PER * 256 / CH;
  constexpr int CPR = CH / kPageSize;   // pieces of a [slot] row
  constexpr int EPP = 16 / EB;          // elements of a piece
  constexpr int ROW = D * EB + 16;      // LDS row
  using E = std::conditional_t<EB == 2, uint16_t, uint8_t>;
  __shared__ __attribute__((aligned(16))) uint8_t tile[BLOCKS][kPageSize][ROW];
  const int H = p.num_kv_heads;
  const int64_t n_blocks = (int64_t)n_pages * H, first = first_page(ids);
  size_t src[PER], dst[PER];  // byte offsets of this thread's pieces
  bool in[PER];
  uint4 kx[PER], vx[PER];
#pragma unroll
  for (int j = 0; j < PER; j++) {
    const int q = threadIdx.x + 256 * j, c = q % CH;
    const int64_t blk = (int64_t)blockIdx.x * BLOCKS + q / CH;
    in[j] = blk < n_blocks;
    const int i = in[j] ? (int)(blk / H) : 0, hd = in[j] ? (int)(blk % H) : 0;
    int page;
    if constexpr (INLINE) page = ids.id[i];
    else page = p.page_ids[i];
    const size_t pool = (((size_t)page * H + hd) * CH + c) * 16, lin = ((size_t)(first * H + blk) * CH + c) * 16;
    src[j] = TO_POOL ? lin : pool;
    dst[j] = TO_POOL ? pool : lin;
    kx[j] = vx[j] = make_uint4(0, 0, 0, 0);
    if (in[j]) {
      kx[j] = load16<!TO_POOL>((const uint8_t*)(TO_POOL ? p.k_lin : p.k_pool) + src[j]);
      vx[j] = load16<!TO_POOL>((const uint8_t*)(TO_POOL ? p.v_lin : p.v_pool) + src[j]);
    }
  }
#pragma unroll
  for (int j = 0; j < PER; j++) {
    if (in[j]) store16<TO_POOL>((uint8_t*)(TO_POOL ? p.k_pool : p.k_lin) + dst[j], kx[j]);
    const int q = threadIdx.x + 256 * j, b = q / CH, c = q % CH;
    if constexpr (TO_POOL) {  // a row piece: slot c / CPR
      *(uint4*)&tile[b][c / CPR][(c % CPR) * 16] = vx[j];
    } else {                  // a column piece: EPP slots of dim d
      const int d = c * EPP / kPageSize, s0 = c * EPP % kPageSize;
      const uint32_t w[4] = {vx[j].x, vx[j].y, vx[j].z, vx[j].w};
#pragma unroll
      for (int e = 0; e < EPP; e++) *(E*)&tile[b][s0 + e][d * EB] = (E)(w[e * EB / 4] >> (8 * EB * e % 32));
    }
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < PER; j++) {
    if (!in[j]) continue;
    const int q = threadIdx.x + 256 * j, b = q / CH, c = q % CH;
    uint4 y;
    if constexpr (TO_POOL) {
      const int d = c * EPP / kPageSize, s0 = c * EPP % kPageSize;
      uint32_t w[4] = {0, 0, 0, 0};
#pragma unroll
      for (int e = 0; e < EPP; e++)
        w[e * EB / 4] |= (uint32_t) * (const E*)&tile[b][s0 + e][d * EB] << (8 * EB * e % 32);
      y = make_uint4(w[0], w[1], w[2], w[3]);
    } else {
      y = *(const uint4*)&tile[b][c / CPR][(c % CPR) * 16];
    }
    store16<TO_POOL>((uint8_t*)(TO_POOL ? p.v_pool : p.v_lin) + dst[j], y);
  }
}

}  // namespace

hipError_t launch_store_kv(const StoreParams& p, int64_t n_units, int head_dim, bool fp8,
                           hipStream_t stream) {
  if (n_units <= 0) return hipSuccess;
  const int hb = head_dim == 128 ? 4 : 8;  // heads per workgroup (HB of the kernel)
  dim3 grid((unsigned)n_units, (unsigned)((p.num_kv_heads + hb - 1) / hb)), block(kStoreThreads);
  if (head_dim == 128) {
    if (fp8) hipLaunchKernelGGL((store_kv_kernel<128, true>), grid, block, 0, stream, p);
    else hipLaunchKernelGGL((store_kv_kernel<128, false>), grid, block, 0, stream, p);
  } else {
    if (fp8) hipLaunchKernelGGL((store_kv_kernel<64, true>), grid, block, 0, stream, p);
    else hipLaunchKernelGGL((store_kv_kernel<64, false>), grid, block, 0, stream, p);
  }
  return hipGetLastError();
}

// Heads per rope workgroup, and the workgroups per page.  Fewer heads give more workgroups,
// more heads compute the page's angles less often.  Measured (us per call, 4 / 8 / 16 /
// 32 heads): 150 pages of 32+8 heads 16.4 / 17.1 / 20.9 / 31.8, 270 pages 24.6 / 22.5 /
// 26.1 / 33.6, 1700 pages of 64+8 heads 255 / 241 / 237 / 246, 2048 pages of 32+8 heads
// 180 / 169 / 157 / 169 -- so up to 2048 workgroups 4 heads, and never more than 16.
// Where all heads of a page are few, one workgroup takes them all once the pages alone fill
// the chip several times: 11000 pages of 8+2 heads of 64 126 us (140 in groups), of 8+1 heads
// of 128 192 us (208); 3000 pages 36.7 us (35.4) and 58.6 us (58.2).
static int64_t rope_groups(RopeParams& p, int64_t n_units) {
  auto log2_up = [](int n) {
    int lg = 0;
    while ((1 << lg) < n) lg++;
    return lg;
  };
  const int Hq = p.num_q_heads, H = p.num_kv_heads;
  p.whole_page = Hq + 2 * H <= 16 && n_units >= 4096;
  p.lg_q = log2_up(Hq);
  p.lg_k = log2_up(H);
  if (p.whole_page) return 1;
  for (int lg = 2;; lg++) {
    // no group larger than the heads there are: its rows past them would idle
    p.lg_q = Hq > 0 ? (lg < log2_up(Hq) ? lg : log2_up(Hq)) : 0;
    p.lg_k = lg < log2_up(H) ? lg : log2_up(H);
    const int64_t groups = (((int64_t)Hq + (1 << p.lg_q) - 1) >> p.lg_q) + (((int64_t)H + (1 << p.lg_k) - 1) >> p.lg_k) +
                           (H + kRopeVHeads - 1) / kRopeVHeads;
    // a grid's y dimension is bounded by 65535 (tens of thousands of heads)
    if (groups <= 65535 && (lg >= 4 || n_units * groups <= 2048)) return groups;
  }
}

hipError_t launch_store_kv_rope(const RopeParams& params, int64_t n_units, int head_dim, bool fp8, bool interleaved,
                                hipStream_t stream) {
  if (n_units <= 0) return hipSuccess;
  RopeParams p = params;
  const int64_t groups = rope_groups(p, n_units);
  dim3 grid((unsigned)n_units, (unsigned)groups), block(kStoreThreads);
#define KVX_ROPE_LAUNCH(D, F, I) hipLaunchKernelGGL((store_kv_rope_kernel<D, F, I>), grid, block, 0, stream, p)
  if (head_dim == 128) {
    if (fp8) { if (interleaved) KVX_ROPE_LAUNCH(128, true, true); else KVX_ROPE_LAUNCH(128, true, false); }
    else { if (interleaved) KVX_ROPE_LAUNCH(128, false, true); else KVX_ROPE_LAUNCH(128, false, false); }
  } else {
    if (fp8) { if (interleaved) KVX_ROPE_LAUNCH(64, true, true); else KVX_ROPE_LAUNCH(64, true, false); }
    else { if (interleaved) KVX_ROPE_LAUNCH(64, false, true); else KVX_ROPE_LAUNCH(64, false, false); }
  }
#undef KVX_ROPE_LAUNCH
  return hipGetLastError();
}

hipError_t launch_page_move(const PageMoveParams& p, int64_t n_pages, hipStream_t stream) {
  if (n_pages <= 0) return hipSuccess;
  hipLaunchKernelGGL(page_move_kernel, dim3((unsigned)n_pages, 2), dim3(256), 0, stream, p);
  return hipGetLastError();
}

template <int D, int EB, bool TO_POOL>
static void launch_page_io_for(const PageIoParams& p, int64_t n_pages, hipStream_t stream) {
  const dim3 block(256);
  constexpr int BLOCKS = 4 * 256 / (D * EB);  // (page, head) blocks per workgroup
  auto grid = [&](int64_t n) { return dim3((unsigned)((n * p.num_kv_heads + BLOCKS - 1) / BLOCKS)); };
  if (p.page_ids != nullptr) {
    hipLaunchKernelGGL((page_io_kernel<D, EB, false, TO_POOL>), grid(n_pages), block, 0, stream, p, (int32_t)n_pages,
                       NoPageIds{});
    return;
  }
  for (int64_t first = 0; first < n_pages; first += kInlinePages) {
    PageIds ids;
    const int64_t n = n_pages - first < kInlinePages ? n_pages - first : kInlinePages;
    ids.first = (int32_t)first;
    for (int64_t i = 0; i < n; i++) ids.id[i] = p.host_ids[first + i];
    hipLaunchKernelGGL((page_io_kernel<D, EB, true, TO_POOL>), grid(n), block, 0, stream, p, (int32_t)n, ids);
  }
}

template <int D, int EB>
static void launch_page_io_dir(const PageIoParams& p, int64_t n_pages, hipStream_t stream) {
  if (p.to_pool) launch_page_io_for<D, EB, true>(p, n_pages, stream);
  else launch_page_io_for<D, EB, false>(p, n_pages, stream);
}

hipError_t launch_page_io(const PageIoParams& p, int64_t n_pages, int head_dim, int elem_bytes,
                          hipStream_t stream) {
  if (n_pages <= 0) return hipSuccess;
  if (head_dim == 128) {
    if (elem_bytes == 2) launch_page_io_dir<128, 2>(p, n_pages, stream);
    else launch_page_io_dir<128, 1>(p, n_pages, stream);
  } else {
    if (elem_bytes == 2) launch_page_io_dir<64, 2>(p, n_pages, stream);
    else launch_page_io_dir<64, 1>(p, n_pages, stream);
  }
  return hipGetLastError();
}

}  // namespace kvx
