// Internal declarations shared by the host code and the HIP kernels of libkvx.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "kvx.h"

namespace kvx {

constexpr int kPageSize = 16;
constexpr int kTileRows = KVX_TILE_ROWS;  // query rows (token x query head of one KV head) per workgroup
constexpr int kTileKeys = 64;   // keys per K/V tile staged in LDS
constexpr int kAttnThreads = 512;  // 8 waves x 32 query rows
constexpr int kNumXcd = 8;      // L2 domains of an MI355X; workgroup i runs on XCD i % 8

// One attention workgroup: a tile of suffix tokens of one request and one KV head,
// over keys [key_begin, key_end) of the request's logical sequence.
struct AttnUnit {
  int32_t qo_row0;    // global suffix row of the tile's first token
  int32_t q_pos0;     // absolute position of that token (P + tok_begin)
  int32_t page_base;  // offset of the request's page list in page_ids
  int32_t key_begin;  // multiple of kTileKeys
  int32_t key_end;    // exclusive; key_end <= key_begin marks a padding entry
  int32_t head_ntok;  // (kv_head << 16) | tokens in the tile (kDecodeUnitFlag: a decode unit)
  int32_t part;       // -1: final result; else index of this part's partial result
  int32_t req;
};
static_assert(sizeof(AttnUnit) == 32, "AttnUnit is 32 bytes");
// In head_ntok of a mixed batch's plan: the unit is one query token over a chunk of its
// keys, run by the decode code (part then counts decode parts).
constexpr int32_t kDecodeUnitFlag = 0x8000;
static_assert(KVX_TILE_ROWS < kDecodeUnitFlag, "tokens of a tile stay below the flag");

// Log-sum-exp merge of the parts of one split tile.
struct MergeUnit {
  int32_t qo_row0;
  int32_t head_ntok;
  int32_t part0;
  int32_t nparts;
};

// One KV-store workgroup: the suffix slots [slot_begin, slot_end) of one page.
struct StoreUnit {
  int32_t row_slot0;  // suffix row that slot 0 of the page would hold (may be negative)
  int32_t page_pos;   // index into page_ids
  int32_t slot_begin;
  int32_t slot_end;
};

// Small plans travel in kernel arguments instead of through a copy (whose start and end
// cost a small call more than its kernels).
//
// Decode: entry e of the arguments stands for `heads` units, unit i being entry i / heads
// with i % heads added to its KV head and (i % heads) times a stride (kept in `req`, which
// no kernel uses) to its part.  heads is 8 where groups of eight units differ in nothing else
// (eight KV heads side by side on the eight XCDs), else 1.
constexpr int kInlineUnits = 110;   // 32-byte units: the arguments stay below 4 KiB
constexpr int kInlineMerges = 220;  // 16-byte merges, one entry for all KV heads of a tile
template <typename U>
struct InlinePlan {
  int32_t n;      // entries; 0: the units are uploaded
  int32_t heads;  // units per entry
  U unit[kInlineUnits];
};
// Prefill: the tiles the units belong to, and a code word per unit, or per `heads` units as
// above.  The kernels that take them are instantiations of their own (kvx_small.hip).
struct PlanTile {
  int32_t qo_row0, q_pos0, page_base;
  int32_t kend;    // keys [0, kend)
  int32_t ntok_nb;  // (tokens << 16) | split boundaries below kend (parts - 1)
  int32_t part0;   // part of (KV head 0, range 0); head h is h * parts further on
};
constexpr int kPlanWords = 960;  // tiles (6 words each), then code words
constexpr uint32_t kPlanPad = 0xFFFFFFFFu;
inline uint32_t plan_code(uint32_t tile, uint32_t head, uint32_t range) { return tile << 20 | head << 10 | range; }
constexpr uint32_t kPlanTiles = 1 << 12, kPlanHeads = 1 << 10, kPlanRanges = 1 << 10;  // limits of the code (tile
                                                                                       // kPlanTiles - 1 is kPlanPad's)
struct CompactPlan {
  int32_t n;        // units
  int32_t n_tiles;
  int32_t heads;    // units per code word
  int32_t split;    // keys per range
  uint32_t words[kPlanWords];
};
template <typename M>
struct InlineMerges {
  int32_t n;      // entries; 0: the merges are uploaded
  int32_t heads;  // merges per entry: KV heads h = 0 .. heads - 1, parts h * nparts further on
  M merge[kInlineMerges];
};

// Unit i of a compact plan whose words are at `words` (constexpr: for the host and the device).
template <class Words>
constexpr AttnUnit unit_from_plan(const CompactPlan& plan, Words words, int i) {
  const uint32_t code = (uint32_t)words[6 * plan.n_tiles + i / plan.heads];
  AttnUnit u{};
  u.part = -1;
  if (code != kPlanPad) {
    const Words t = words + 6 * (code >> 20);
    const int h = (int)(code >> 10 & (kPlanHeads - 1)) + i % plan.heads, range = (int)(code & (kPlanRanges - 1));
    const int ntok = (int)t[4] >> 16, nb = (int)t[4] & 0xFFFF;
    u.qo_row0 = (int)t[0];
    u.q_pos0 = (int)t[1];
    u.page_base = (int)t[2];
    u.key_begin = range * plan.split;
    u.key_end = range < nb ? (range + 1) * plan.split : (int)t[3];
    u.head_ntok = h << 16 | ntok;
    if (nb > 0) u.part = (int)t[5] + h * (nb + 1) + range;
  }
  return u;
}

struct AttnParams {
  const uint16_t* q;      // bf16 [T, Hq, D]
  uint16_t* out;          // bf16 [T, Hq, D]
  float* lse;             // fp32 [T, Hq] or null
  const void* k_pool;
  const void* v_pool;
  const int32_t* page_ids;
  const AttnUnit* units;
  float* o_part;          // fp32 [parts, kTileRows * D], in the accumulators' order (write_result)
  float* lse_part;        // fp32 [parts, kTileRows]
  const float* k_scale;   // fp8 pool: device [Hkv]
  const float* v_scale;
  int32_t num_q_heads;
  int32_t num_kv_heads;
  int32_t group;          // Hq / Hkv
  int32_t tile_tok;       // tokens per tile = kTileRows / group
  float scale_log2;       // sm_scale * log2(e)
  int32_t mixed;          // 1: the plan holds decode units too
  float* d_part;          // fp32 [decode parts, kDecodeMaxGroup, D]
  float* d_lse;           // fp32 [decode parts, kDecodeMaxGroup]
  // For the launcher: the plan (in host memory) for the kernel arguments, or null when the
  // units were uploaded.
  const CompactPlan* compact;
};

struct MergeParams {
  const MergeUnit* merges;
  const float* o_part;
  const float* lse_part;
  uint16_t* out;
  float* lse;
  int32_t num_q_heads;
  int32_t group;
  InlineMerges<MergeUnit> plan;  // plan.n > 0: the merges
};
static_assert(sizeof(MergeParams) <= 4096, "kernel arguments");

// The requests of a small store batch, passed by value in the kernel arguments so
// that no unit list is uploaded: request r's pages are the workgroups
// [first[r], first[r + 1]), logical pages prefix[r] / 16 onwards.
constexpr int kStoreInlineReqs = 96;
struct StoreReqs {
  int32_t n;                            // requests with work; 0: use the uploaded unit list
  int32_t first[kStoreInlineReqs + 1];  // first workgroup of each request; first[n] = all
  int32_t qo[kStoreInlineReqs];         // suffix row of the request's first suffix token
  int32_t prefix[kStoreInlineReqs];     // P
  int32_t end[kStoreInlineReqs];        // P + E
  int32_t page_base[kStoreInlineReqs];  // page_indptr[r]
};

struct StoreParams {
  const uint16_t* k_ext;  // bf16 [T, Hkv, D]
  const uint16_t* v_ext;
  void* k_pool;
  void* v_pool;
  const int32_t* page_ids;
  const StoreUnit* units;
  const float* k_inv_scale;  // fp8 pool: device [Hkv], fp32 1/scale
  const float* v_inv_scale;
  int32_t num_kv_heads;
  StoreReqs reqs;            // reqs.n > 0: the units come from here instead
};

// One fused-store workgroup: a StoreUnit plus the absolute position of slot 0.
struct RopeUnit {
  int32_t row_slot0;
  int32_t page_pos;
  int32_t slot_begin;
  int32_t slot_end;
  int32_t pos_slot0;  // position t of slot 0 of the page (a multiple of 16)
};

constexpr int kRopeMaxPlanes = 64;  // rotary_dim / 2 <= head_dim / 2

struct RopeParams {
  const uint16_t* q;      // bf16 [T, Hq, D], or null when num_q_heads == 0
  uint16_t* q_out;        // may equal q
  const uint16_t* k_ext;  // bf16 [T, Hkv, D]
  const uint16_t* v_ext;
  void* k_pool;
  void* v_pool;
  const int32_t* page_ids;
  const RopeUnit* units;
  const float* k_inv_scale;  // fp8 pool: device [Hkv], fp32 1/scale
  const float* v_inv_scale;
  const uint16_t* q_norm;    // bf16 [D] RMS-norm weights, or null
  const uint16_t* k_norm;
  int32_t num_q_heads;
  int32_t num_kv_heads;
  int32_t rotary_dim;        // multiple of 16, <= D
  float norm_eps;
  // set by the launcher: log2 of the Q and of the K heads per workgroup, and whether one
  // workgroup takes all heads of a page
  int32_t lg_q;
  int32_t lg_k;
  int32_t whole_page;
  double rev_freq[kRopeMaxPlanes];  // plane rate in revolutions per position: f_j / (2 pi)
  StoreReqs reqs;                   // reqs.n > 0: the units come from here instead
};

// Page ids of one launch of the page I/O kernel in its arguments.
constexpr int kInlinePages = 960;
struct PageIoParams {
  const int32_t* page_ids;  // device [n], or null: host_ids
  const int32_t* host_ids;  // for the launcher: host [n], carried in kernel arguments
  void* k_pool;
  void* v_pool;
  void* k_lin;              // canonical [n][Hkv][16][D] buffers
  void* v_lin;
  int32_t num_kv_heads;
  int32_t to_pool;          // 1: write pages into the pool, 0: read them out
};

// Raw page records between the pool and host memory: record i = the K block then
// the V block of page page_ids[i], at host + slots[i] * 2 * block_bytes.
struct PageMoveParams {
  const int32_t* page_ids;  // device [n]
  const int32_t* slots;     // device [n]
  uint8_t* k_pool;
  uint8_t* v_pool;
  uint8_t* host;            // device-accessible address of pinned host memory
  int64_t block_bytes;      // Hkv * 16 * D * elem bytes (a multiple of 1 KiB)
  int32_t to_host;          // 1: pool -> host (spill), 0: host -> pool (reload)
};

// ---- decode (one query token per request): a key chunk of one (request, KV head)
constexpr int kDecodeThreads = 256;  // 4 waves, each streaming every 4th pair of pages
constexpr int kDecodeMaxGroup = 16;  // query heads per KV head held in one MFMA column block
constexpr int kDecodeChunkAlign = 64;  // chunk boundaries are multiples of it (keys)

struct DecodeUnit {
  int32_t qo_row;     // the request's only suffix row
  int32_t page_base;  // offset of the request's page list in page_ids
  int32_t key_begin;  // multiple of kDecodeChunkAlign
  int32_t key_end;    // exclusive
  int32_t head;       // KV head
  int32_t part;       // -1: final result; else index of this chunk's partial result
  int32_t req;
  int32_t pad;
};
static_assert(sizeof(DecodeUnit) == 32, "DecodeUnit is 32 bytes");

struct DecodeMerge {
  int32_t qo_row;
  int32_t head;
  int32_t part0;
  int32_t nparts;
};

struct DecodeArgs {
  const uint16_t* q;      // bf16 [T, Hq, D]
  uint16_t* out;          // bf16 [T, Hq, D]
  float* lse;             // fp32 [T, Hq] or null
  const void* k_pool;     // [page][kv_head][slot][D], bf16 or fp8
  const void* v_pool;     // [page][kv_head][D][slot]
  const int32_t* page_ids;
  float* o_part;          // fp32 [parts, kDecodeMaxGroup, D]
  float* lse_part;        // fp32 [parts, kDecodeMaxGroup]
  const float* k_scale;   // fp8 pool: device [Hkv]
  const float* v_scale;
  int32_t num_q_heads;
  int32_t num_kv_heads;
  int32_t group;          // Hq / Hkv <= kDecodeMaxGroup
  float scale_log2;
};

// Page lists of the requests that decode in a batch read with non-temporal loads, to tell
// pages that several of them hold from a request's own: list i is page_ids[base[i]] up to
// base[i + 1].
constexpr int kShareReqs = 256;
struct DecodeLists {
  const int32_t* base;               // device [n + 1], or null: in_args
  int32_t n;                         // 0: plain loads throughout
  int32_t in_args[kInlineUnits + 1];
};

struct DecodeParams {
  DecodeArgs a;
  const DecodeUnit* units;
  DecodeLists lists;
  InlinePlan<DecodeUnit> plan;  // plan.n > 0: the units (and lists.in_args the lists)
};
static_assert(sizeof(DecodeParams) <= 4096, "kernel arguments");

struct DecodeMergeParams {
  const DecodeMerge* merges;
  const float* o_part;
  const float* lse_part;
  uint16_t* out;
  float* lse;
  int32_t num_q_heads;
  int32_t group;
  InlineMerges<DecodeMerge> plan;  // plan.n > 0: the merges
};
static_assert(sizeof(DecodeMergeParams) <= 4096, "kernel arguments");

hipError_t launch_decode(const DecodeParams& p, int64_t n_units, int head_dim, bool fp8, hipStream_t stream);
hipError_t launch_decode_merge(const DecodeMergeParams& p, int64_t n_merges, int head_dim, hipStream_t stream);

// Record a failure for kvx_last_error() and return `code` (host code of any file).
int report(int code, const char* fmt, ...) __attribute__((format(printf, 2, 3)));

// Fixed device scratch of the allocation-free attention entry point: a plan region
// of plan_bytes followed by a partial-result region of parts_bytes, at an address
// that `address` gives per device (called with that device current).
struct FixedScratch {
  size_t plan_bytes;
  size_t parts_bytes;
  int (*address)(int device, void** base);
};

// extend_attention's whole call: argument checks, plan, upload, launches.  With
// fixed == nullptr a plan too large for the kernel arguments goes through the pool's
// staging buffer and split parts into its growable workspace; otherwise both go into
// the fixed scratch, the plan is bounded by its regions (EUNSUPPORTED beyond them, checked on the
// host before any device call) and nothing is allocated.
int attention_call(kvx_pool* pool, const kvx_batch* batch, const void* q, int32_t num_q_heads, float sm_scale,
                   void* out, float* lse, kvx_stream_t stream, const FixedScratch* fixed);

hipError_t launch_extend_attention(const AttnParams& p, int64_t n_units, int head_dim, bool fp8, bool scaled_q,
                                   hipStream_t stream);
// launch_extend_attention of a plan that holds decode units (p.mixed)
hipError_t launch_mixed_attention(const AttnParams& p, int64_t n_units, int head_dim, bool fp8, bool scaled_q,
                                  hipStream_t stream);
// ... and of a compact plan, from the kernel arguments
hipError_t launch_small_attention(const AttnParams& p, int64_t n_units, int head_dim, bool fp8, bool scaled_q,
                                  hipStream_t stream);
hipError_t launch_merge(const MergeParams& p, int64_t n_merges, int head_dim, hipStream_t stream);
hipError_t launch_store_kv(const StoreParams& p, int64_t n_units, int head_dim, bool fp8,
                           hipStream_t stream);
hipError_t launch_store_kv_rope(const RopeParams& p, int64_t n_units, int head_dim, bool fp8, bool interleaved,
                                hipStream_t stream);
hipError_t launch_page_move(const PageMoveParams& p, int64_t n_pages, hipStream_t stream);
hipError_t launch_page_io(const PageIoParams& p, int64_t n_pages, int head_dim, int elem_bytes,
                          hipStream_t stream);

}  // namespace kvx
