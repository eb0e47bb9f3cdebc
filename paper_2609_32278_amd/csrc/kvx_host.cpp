// Host side of libkvx: the C ABI declared in include/kvx.h.
//
// Owns the KV pool (hipMalloc), checks every argument before queuing work,
// plans extend_attention's work over ragged (prefix_len, extend_len) pairs and
// passes the plan in kernel arguments where it is small, else uploads it through
// pinned staging buffers on the caller's stream.

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <numeric>
#include <queue>
#include <string>
#include <utility>
#include <vector>

#include "kvx_internal.h"

using kvx::AttnUnit;
using kvx::MergeUnit;
using kvx::StoreUnit;

namespace {

thread_local std::string g_last_error;

int fail(int code, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  g_last_error = buf;
  return code;
}

}  // namespace

int kvx::report(int code, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  g_last_error = buf;
  return code;
}

namespace {

int hip_fail(hipError_t e, const char* what) {
  return fail(e == hipErrorOutOfMemory ? KVX_ENOMEM : KVX_EHIP, "%s: %s", what, hipGetErrorString(e));
}

#define KVX_HIP(call)                                   \
  do {                                                  \
    hipError_t e_ = (call);                             \
    if (e_ != hipSuccess) return hip_fail(e_, #call);   \
  } while (0)

bool validate_mode() {
  const char* v = std::getenv("KVX_VALIDATE");
  return v != nullptr && v[0] != '\0' && v[0] != '0';
}

// Pinned host buffer + device buffer + events: a reusable upload channel.  The
// host side is rewritten only after the previous copy out of it has completed.
// The device buffer grows with the stream-ordered allocator: the old buffer is
// freed in stream order behind `used` (recorded after the last kernels that read
// it), so growing never waits on the host for the device.
struct Staging {
  void* host = nullptr;
  size_t host_cap = 0;
  void* dev = nullptr;
  size_t dev_cap = 0;
  hipEvent_t ev = nullptr;    // after the last copy out of `host`
  hipEvent_t used = nullptr;  // after the last kernels that read `dev`
  bool pending = false;

  // Only after the device has gone idle (pool destruction).
  void release() {
    if (ev) {
      (void)hipEventSynchronize(ev);
      (void)hipEventDestroy(ev);
    }
    if (used) (void)hipEventDestroy(used);
    if (host) (void)hipHostFree(host);
    if (dev) (void)hipFreeAsync(dev, nullptr);
    *this = Staging();
  }

  // Copy `bytes` from `src` to device memory ordered on `stream`; *out receives the
  // device address (valid until the next upload on this channel is ordered after it).
  // The caller records done() on the stream after the kernels that read it.
  int upload(const void* src, size_t bytes, hipStream_t stream, void** out) {
    if (!ev) KVX_HIP(hipEventCreateWithFlags(&ev, hipEventDisableTiming));
    if (!used) KVX_HIP(hipEventCreateWithFlags(&used, hipEventDisableTiming));
    if (pending) {
      KVX_HIP(hipEventSynchronize(ev));
      pending = false;
    }
    if (bytes > host_cap) {
      if (host) KVX_HIP(hipHostFree(host));
      host = nullptr;
      size_t cap = std::max<size_t>(bytes + bytes / 2, 4096);
      KVX_HIP(hipHostMalloc(&host, cap, hipHostMallocDefault));
      host_cap = cap;
    }
    if (bytes > dev_cap) {
      if (dev) {
        // earlier kernels (on any stream) that read the old buffer precede `used`
        KVX_HIP(hipStreamWaitEvent(stream, used, 0));
        KVX_HIP(hipFreeAsync(dev, stream));
      }
      dev = nullptr;
      dev_cap = 0;
      size_t cap = std::max<size_t>(bytes + bytes / 2, 4096);
      KVX_HIP(hipMallocAsync(&dev, cap, stream));
      dev_cap = cap;
    }
    std::memcpy(host, src, bytes);
    KVX_HIP(hipMemcpyAsync(dev, host, bytes, hipMemcpyHostToDevice, stream));
    KVX_HIP(hipEventRecord(ev, stream));
    pending = true;
    *out = dev;
    return KVX_OK;
  }

  int done(hipStream_t stream) {
    KVX_HIP(hipEventRecord(used, stream));
    return KVX_OK;
  }
};

// Device scratch that only grows, with the same stream-ordered replacement.
struct Workspace {
  void* ptr = nullptr;
  size_t cap = 0;
  hipEvent_t used = nullptr;  // after the last kernels that used `ptr`
  int ensure(size_t bytes, hipStream_t stream) {
    if (!used) KVX_HIP(hipEventCreateWithFlags(&used, hipEventDisableTiming));
    if (bytes <= cap) return KVX_OK;
    if (ptr) {
      KVX_HIP(hipStreamWaitEvent(stream, used, 0));
      KVX_HIP(hipFreeAsync(ptr, stream));
      ptr = nullptr;
      cap = 0;
    }
    // headroom of a quarter for small sizes; past 1 GiB exactly what is asked
    size_t c = bytes > ((size_t)1 << 30) ? bytes : std::max<size_t>(bytes + bytes / 4, 1 << 20);
    KVX_HIP(hipMallocAsync(&ptr, c, stream));
    cap = c;
    return KVX_OK;
  }
  int done(hipStream_t stream) {
    if (used) KVX_HIP(hipEventRecord(used, stream));
    return KVX_OK;
  }
  // Only after the device has gone idle (pool destruction).
  void release() {
    if (ptr) (void)hipFreeAsync(ptr, nullptr);
    if (used) (void)hipEventDestroy(used);
    ptr = nullptr;
    cap = 0;
    used = nullptr;
  }
};

constexpr int kPlanSlots = 256;  // 256 CUs x 1 resident attention workgroup
// Bound on the partial results of split key ranges: 16384 parts x 256 rows x 128
// dims x 4 B = 2 GiB (+16 MiB of LSE) at head_dim 128, allocated exactly.
constexpr int64_t kMaxParts = 16384;

}  // namespace

struct kvx_pool {
  int device = 0;
  int64_t num_pages = 0;
  int32_t page_size = 16;
  int32_t num_kv_heads = 0;
  int32_t head_dim = 0;
  int32_t kv_dtype = KVX_KV_BF16;
  int32_t elem_bytes = 2;
  void* k = nullptr;
  void* v = nullptr;
  float* scales_d = nullptr;  // [k_scale | v_scale | k_inv | v_inv], each num_kv_heads
  Staging st_store, st_attn, st_io, st_move;
  Workspace parts;
  int32_t split_keys = 0;  // key-range split length of extend_attention; 0 = automatic
  int32_t scaled_q = 0;    // 1: prefill attention on a bf16 pool takes the folded softmax
};

namespace {

int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

int check_pool(const kvx_pool* pool) {
  if (pool == nullptr) return fail(KVX_EINVAL, "pool is NULL");
  return KVX_OK;
}

// The kernels move 16-byte pieces: every bf16 row buffer must start 16-byte aligned.
int check_align(const void* ptr, const char* name) {
  if (ptr != nullptr && ((uintptr_t)ptr & 15u) != 0)
    return fail(KVX_EINVAL, "%s = %p is not 16-byte aligned", name, ptr);
  return KVX_OK;
}

int use_device(const kvx_pool* pool) {
  int cur = -1;
  KVX_HIP(hipGetDevice(&cur));
  if (cur != pool->device) KVX_HIP(hipSetDevice(pool->device));
  return KVX_OK;
}

// Host-side checks of a batch; fills qo offsets (request r owns rows [qo[r], qo[r+1])).
int check_batch(const kvx_batch* b, std::vector<int64_t>& qo, bool need_page_ids = true) {
  if (b == nullptr) return fail(KVX_EINVAL, "batch is NULL");
  if (b->num_reqs < 0) return fail(KVX_EINVAL, "num_reqs = %d < 0", b->num_reqs);
  qo.assign((size_t)b->num_reqs + 1, 0);
  if (b->num_reqs == 0) return KVX_OK;
  if (!b->prefix_lens || !b->extend_lens || !b->page_indptr)
    return fail(KVX_EINVAL, "prefix_lens, extend_lens and page_indptr must be non-NULL");
  if (b->page_indptr[0] != 0) return fail(KVX_EINVAL, "page_indptr[0] = %d, must be 0", b->page_indptr[0]);
  for (int r = 0; r < b->num_reqs; r++) {
    const int64_t P = b->prefix_lens[r], E = b->extend_lens[r];
    if (P < 0 || E < 0) return fail(KVX_EINVAL, "request %d: negative length (P=%lld, E=%lld)", r, (long long)P, (long long)E);
    if (P + E > (int64_t)INT32_MAX - 1024) return fail(KVX_EINVAL, "request %d: sequence too long", r);
    const int64_t have = (int64_t)b->page_indptr[r + 1] - b->page_indptr[r];
    if (have < ceil_div(P + E, kvx::kPageSize))
      return fail(KVX_EINVAL, "request %d: %lld page ids for %lld tokens (need %lld)", r, (long long)have,
                  (long long)(P + E), (long long)ceil_div(P + E, kvx::kPageSize));
    qo[r + 1] = qo[r] + E;
  }
  if (qo.back() > (int64_t)INT32_MAX) return fail(KVX_EINVAL, "total extend length exceeds 2^31-1");
  if (need_page_ids && b->page_indptr[b->num_reqs] > 0 && b->page_ids == nullptr)
    return fail(KVX_EINVAL, "page_ids is NULL");
  return KVX_OK;
}

// KVX_VALIDATE=1: copy the page table to the host and check every id.
int check_page_ids(const kvx_pool* pool, const kvx_batch* b, hipStream_t stream) {
  const int64_t n = b->num_reqs ? b->page_indptr[b->num_reqs] : 0;
  if (n == 0) return KVX_OK;
  std::vector<int32_t> ids((size_t)n);
  KVX_HIP(hipStreamSynchronize(stream));
  KVX_HIP(hipMemcpy(ids.data(), b->page_ids, (size_t)n * sizeof(int32_t), hipMemcpyDeviceToHost));
  for (int64_t i = 0; i < n; i++)
    if (ids[(size_t)i] < 0 || ids[(size_t)i] >= pool->num_pages)
      return fail(KVX_ERANGE, "page_ids[%lld] = %d outside [0, %lld)", (long long)i, ids[(size_t)i],
                  (long long)pool->num_pages);
  return KVX_OK;
}

struct Plan {
  std::vector<AttnUnit> units;  // in launch order (position i runs on XCD i % 8)
  std::vector<MergeUnit> merges;
  bool inspect = false;              // fill items: the same units in the same order, for
  std::vector<kvx_work_item> items;  // extend_attention_plan
  int64_t n_parts = 0;
  std::vector<kvx::PlanTile> tiles;  // what the units are made of, and a code word each
  std::vector<uint32_t> codes;       // (empty if the batch is beyond their limits)
  int64_t split = 0;
  // decode units among the units (mixed batches)
  bool mixed = false;
  std::vector<kvx::DecodeMerge> dec_merges;
  int64_t dec_parts = 0;
};

// Bounds on the partial results of a plan.
struct PartLimits {
  int64_t prefill, decode;
};
// Those of a call on the pool's workspace: the rows of kMaxParts tiles in all, decode parts
// counting a sixteenth.
static_assert(kvx::kTileRows == 16 * kvx::kDecodeMaxGroup, "rows of a part");
constexpr PartLimits pool_limits(bool mixed) {
  return PartLimits{mixed ? kMaxParts - kMaxParts / 16 : kMaxParts, kMaxParts};
}

// A tile of suffix tokens of one request; every KV head has the same tiles.
struct Tile {
  int32_t r, tok0, ntok;
  int64_t kend, qpos0;  // keys [0, kend); position of the first token
};

// What a unit costs besides its iterations over 64 keys, in such iterations (about 1.7 us
// at head_dim 128 on a busy chip, 0.9 us at 64): its first loads and its epilogue; the
// fp32 result of a part of 256 rows, written and read again; the merge launch.  Set so
// that the split chosen below is the fastest one or nearly: on 13 batches timed with 12 forced
// split lengths each, within 2% of the best in calls above 500 us and 1-6%, the search's own
// host time with it, below (units alone take 11.5 and 8.0 us for one tile).
struct UnitCosts {
  double start, part, merge;
};
constexpr UnitCosts kUnitCosts128{8.0, 4.0, 3.0}, kUnitCosts64{11.0, 4.0, 3.0};

// Decode units of a mixed batch, in the same measure: 64 keys stream in about 0.4
// iterations.
constexpr double kDecodePerIter = 0.4;
// Share of them spread evenly over the prefill units, which they overlap; the rest fill up
// the end.  3 prefilling requests with 61 decoding ones (1k-16k contexts, 32/8/128 heads): 604 us
// a call, 613 us with three quarters, 638 us with all of them spread, 680 us with all at the
// end.  Against tiles for all, 23 mixes (1-8 prefilling, 4-96 decoding, head_dim 64 and 128,
// both pool types) take 0.48-0.97 of the time.
constexpr double kDecodeSpread = 0.6;
struct Filler {
  int64_t units = 0;  // of one KV head
  double cost = 0.0;  // of one unit
};

// The trial schedules of one search: one KV head's units on its share of the 256 workgroup
// slots.  Planning is on the path of every call, so a trial keeps its memory, takes equal
// units and equal slots as groups, and gives up once it cannot be the shortest (24 requests of
// 124-239 tokens on 8/1/128 heads, 148 tiles: 500 -> 58 us a plan).
class Trials {
 public:
  Trials(const std::vector<Tile>& tiles, int32_t Hkv, int32_t tile_tok, const UnitCosts& k, const Filler& filler)
      : tiles_(tiles), tile_tok_(tile_tok), slots_(std::max<int64_t>(1, kPlanSlots / Hkv)), k_(k), filler_(filler) {}

  // The units when key ranges are split every `split` keys (0 = not at all): returns the
  // number of parts.
  int64_t cut(int64_t split) {
    const int BN = kvx::kTileKeys;
    units_.clear();
    total_ = 0.0;
    auto add = [&](double c, int64_t n) {
      total_ += c * (double)n;
      if (!units_.empty() && units_.back().first == c) units_.back().second += n;
      else units_.push_back({c, n});
    };
    parts_ = 0;
    int64_t inner = 0;  // inner parts of whole tiles, all alike
    int64_t nb = 0;     // boundaries split, 2 split, ... <= qpos0
    for (size_t i = 0; i < tiles_.size(); i++) {
      const Tile& t = tiles_[i];
      // a request's tiles come longest first, a few tokens apart
      if (split > 0 && (i == 0 || t.r != tiles_[i - 1].r)) nb = t.qpos0 / split;
      while (nb * split > t.qpos0) nb--;
      const double extra = nb > 0 ? k_.start + k_.part * t.ntok / tile_tok_ : k_.start;
      if (nb > 0) {
        if (t.ntok == tile_tok_) inner += nb;
        else add((double)(split / BN) + extra, nb);
        parts_ += nb + 1;
      }
      add((double)ceil_div(t.kend - nb * split, BN) + extra, 1);
    }
    if (inner > 0) add((double)(split / BN) + (k_.start + k_.part * tile_tok_ / tile_tok_), inner);
    if (filler_.units > 0) {
      total_ += filler_.cost * (double)filler_.units;
      units_.push_back({filler_.cost, filler_.units});
    }
    return parts_;
  }

  // Duration, in iterations, of the longest-first schedule of these units with the merge
  // launch; or any value of at least `cap` if it is no shorter than that.
  double length(double cap) {
    const double merge = parts_ > 0 ? k_.merge : 0.0;
    const double even = total_ / (double)slots_ * (1.0 - 1e-9);
    if (even + merge >= cap) return even + merge;
    std::sort(units_.begin(), units_.end(), [](const auto& x, const auto& y) { return x.first > y.first; });
    // slots as groups of equal load, a heap with the least loaded first
    heap_.assign(1, {0.0, slots_});
    double end = 0.0;
    for (auto [cost, n] : units_) {
      while (n > 0) {
        const auto [load, count] = heap_[0];
        const int64_t m = std::min(n, count);
        end = std::max(end, load + cost);
        if (end + merge >= cap) return end + merge;
        sink({load + cost, m});
        if (count > m) rise({load, count - m});
        n -= m;
      }
    }
    return end + merge;
  }

 private:
  typedef std::pair<double, int64_t> Group;  // cost or load, how many
  void sink(Group g) {  // in place of the first
    size_t i = 0;
    for (size_t c; (c = 2 * i + 1) < heap_.size(); i = c) {
      if (c + 1 < heap_.size() && heap_[c + 1].first < heap_[c].first) c++;
      if (g.first <= heap_[c].first) break;
      heap_[i] = heap_[c];
    }
    heap_[i] = g;
  }
  void rise(Group g) {
    size_t i = heap_.size();
    heap_.push_back(g);
    for (size_t up; i > 0 && heap_[up = (i - 1) / 2].first > g.first; i = up) heap_[i] = heap_[up];
    heap_[i] = g;
  }

  const std::vector<Tile>& tiles_;
  const int32_t tile_tok_;
  const int64_t slots_;
  const UnitCosts k_;
  const Filler filler_;
  std::vector<Group> units_, heap_;
  double total_ = 0.0;
  int64_t parts_ = 0;
};

// Length (keys, a multiple of 64) of the parts key ranges are split into, 0 = no split.
//   * A batch whose longest tile is at most an eighth of a slot's share of the work runs
//     unsplit, and so does one whose unsplit schedule is within 4% of perfect balance.
//   * Otherwise the schedule is worked out for no split, for the shortest parts that give
//     one and two units per slot, and for lengths in steps of 1.3 from 1.5 times a slot's
//     share to a fifth of it; the shortest schedule wins, the last ones only by 3% (a
//     200000-token prefix under 300 tokens: 1713 us in two whole rounds, 1694 us in five).
//     One of a single round of parts counts 6% of a part more: it ends with its slowest CU
//     (the XCDs' clocks differ by 4-7%) and has no shorter unit to even that out.  Parts
//     have at least 4 iterations.
//   * Where one of these has more than max_parts parts, the shortest length that keeps within
//     them and ten longer ones in steps of 1.1 are tried too (the allocation-free call holds
//     about 420 parts at head_dim 128: 3 requests of 313-494 tokens on about 40000 each, 32/8
//     heads, 911 us without these and 788 with).
int64_t choose_split(const std::vector<Tile>& tiles, int32_t Hkv, int32_t tile_tok, int32_t D, const Filler& filler,
                     int64_t max_parts) {
  const int BN = kvx::kTileKeys;
  const UnitCosts& k = D == 128 ? kUnitCosts128 : kUnitCosts64;
  int64_t total = 0, longest = 0;
  for (const Tile& t : tiles) {
    const int64_t c = ceil_div(t.kend, BN);
    total += c;
    longest = std::max(longest, c);
  }
  const double slots = std::max(1.0, (double)kPlanSlots / Hkv);  // per KV head
  const double share = ((double)total + filler.cost * (double)filler.units) / slots;  // iterations per slot
  if ((double)longest * 8 <= share) return 0;
  constexpr double kNever = 1e300;
  Trials trial(tiles, Hkv, tile_tok, k, filler);
  trial.cut(0);
  int64_t best_split = 0;
  double best = trial.length(kNever);
  if (best <= 1.04 * (share + k.start * std::max(1.0, (double)tiles.size() / slots))) return 0;
  auto units_at = [&](int64_t len) {  // iterations per part; the count never grows with it
    const int64_t split = len * BN;
    int64_t n = 0, nb = 0;
    for (size_t i = 0; i < tiles.size(); i++) {
      const int64_t q = tiles[i].qpos0;
      if (i == 0 || tiles[i].r != tiles[i - 1].r) nb = q / split;
      while (nb * split > q) nb--;
      n += nb + 1;
    }
    return n;
  };
  bool refused = false;  // a length was, for its parts
  auto try_length = [&](int64_t len, double margin) {
    if (((double)len + k.merge) * margin >= best) return;  // cannot win
    const int64_t parts = trial.cut(len * BN);
    refused |= parts * Hkv > max_parts;
    if (parts == 0 || parts * Hkv > max_parts) return;
    const double one_round = (double)parts <= slots ? 0.06 * (double)len : 0.0;
    const double t = (trial.length(best / margin * (1.0 + 1e-9) - one_round) + one_round) * margin;
    if (t < best) {
      best = t;
      best_split = len * BN;
    }
  };
  double keys = 0.0;
  for (const Tile& t : tiles) keys += (double)t.qpos0;
  for (const int rounds : {1, 2}) {
    // the shortest parts of at most this many units; a tile has more than qpos0 / part and
    // at most qpos0 / part + 1
    const double most = rounds * slots, rest = most - (double)tiles.size();
    int64_t lo = std::min(longest, std::max<int64_t>(4, (int64_t)(keys / BN / most)));
    int64_t hi = rest > 0 ? std::min<int64_t>(longest, std::max<int64_t>(4, (int64_t)(keys / BN / rest) + 2)) : longest;
    hi = std::max(lo, hi);
    while (lo < hi) {
      const int64_t mid = lo + (hi - lo) / 2;
      if ((double)units_at(mid) <= most) hi = mid;
      else lo = mid + 1;
    }
    try_length(lo, 1.0);
  }
  double len = std::min((double)longest / 2, 1.5 * share);
  for (int i = 0; i < 10 && len >= std::max(4.0, share / 5); i++, len /= 1.3) try_length((int64_t)len, 1.03);
  if (refused) {
    int64_t lo = 4, hi = longest;  // the number of parts never grows with their length
    while (lo < hi) {
      const int64_t mid = lo + (hi - lo) / 2;
      if (trial.cut(mid * BN) * Hkv <= max_parts) hi = mid;
      else lo = mid + 1;
    }
    for (int i = 0; i <= 10 && lo < longest; i++, lo += (lo + 9) / 10) try_length(lo, 1.0);
  }
  return best_split;
}

// Whether the one-token suffixes of a batch become decode units next to the tiles of the
// longer ones: when through tiles they would take a slot at least 8 iterations (below
// that the merge of their chunks costs what they save).
bool is_mixed_batch(const kvx_batch* b, int32_t Hq, int32_t Hkv) {
  int64_t one_token = 0;  // iterations, all KV heads
  for (int r = 0; r < b->num_reqs; r++)
    if (b->extend_lens[r] == 1) one_token += Hkv * ceil_div((int64_t)b->prefix_lens[r] + 1, kvx::kTileKeys);
  return Hq / Hkv <= kvx::kDecodeMaxGroup && one_token >= 8 * kPlanSlots;
}

// Work plan of extend_attention.
//   * every request's suffix is cut into tiles of tile_tok tokens (x group query heads
//     = 256 rows) per KV head; a tile covers keys [0, P + last token of the tile];
//   * key ranges may be split at multiples of the tile width into parts, merged by
//     log-sum-exp afterwards (choose_split);
//   * each (request, KV head) is bound to one XCD (KV head h -> XCD h % 8 when the
//     head count is a multiple of 8), so the workgroups that stream the same K/V
//     pages share one L2; for other head counts each (request, KV head, part of a
//     split key range) is bound greedily by cost, so that a batch of few long
//     requests still spreads its parts over all eight XCDs (the parts of one key
//     range, read by every tile of the request, stay together);
//   * within an XCD, the units of a split batch, or of one of less than four rounds, go
//     longest first, those over one key range next to each other.  Other batches keep
//     each request together instead, requests by their longest tile and tiles longest
//     first, which is nearly longest first and streams one request's pages at a time.  (By
//     total work of the request, a request of few long tiles came last: 16 agents with
//     4k-32k prefixes, 3.19 -> 2.85 ms.)
//   * mixed: one-token suffixes become decode units, key chunks of the (request, KV head).
//   * packed: the smallest plan there is, without padding and with no split but a forced one; a
//     unit then runs on whatever XCD its place gives it.
int make_plan(const kvx_batch* b, const std::vector<int64_t>& qo, int32_t Hq, int32_t Hkv, int32_t D,
              int32_t split_keys, const PartLimits& limits, bool mixed, Plan& plan, bool packed = false) {
  const int G = Hq / Hkv;
  const int tile_tok = kvx::kTileRows / G;
  const int BN = kvx::kTileKeys;

  plan.mixed = mixed;
  // requests by their longest tile
  std::vector<int32_t> order;
  for (int r = 0; r < b->num_reqs; r++)
    if (b->extend_lens[r] > (plan.mixed ? 1 : 0)) order.push_back(r);
  std::stable_sort(order.begin(), order.end(), [&](int32_t x, int32_t y) {
    return (int64_t)b->prefix_lens[x] + b->extend_lens[x] > (int64_t)b->prefix_lens[y] + b->extend_lens[y];
  });
  std::vector<Tile> tiles;  // request by request, a request's longest tile first
  for (const int32_t r : order) {
    const int64_t P = b->prefix_lens[r], E = b->extend_lens[r];
    for (int64_t t0 = (E - 1) / tile_tok * tile_tok; t0 >= 0; t0 -= tile_tok) {
      const int64_t ntok = std::min<int64_t>(tile_tok, E - t0);
      tiles.push_back(Tile{r, (int32_t)t0, (int32_t)ntok, P + t0 + ntok, P + t0});
    }
  }

  // decode units: chunks of 2048 keys (long enough to hide their start, short enough to
  // fill gaps), shorter where that leaves fewer than 512
  Filler filler;
  int64_t chunk = 0;
  std::vector<AttnUnit> dec_units;
  plan.dec_merges.clear();
  plan.dec_parts = 0;
  if (plan.mixed) {
    const int64_t A = kvx::kDecodeChunkAlign;
    int64_t one_keys = 0;  // keys of one-token suffixes, all KV heads
    for (int r = 0; r < b->num_reqs; r++)
      if (b->extend_lens[r] == 1) one_keys += Hkv * ((int64_t)b->prefix_lens[r] + 1);
    chunk = split_keys > 0 ? split_keys : std::min<int64_t>(2048, std::max<int64_t>(512, one_keys / 512)) / A * A;
    auto chunks_of = [&](int r) { return ceil_div((int64_t)b->prefix_lens[r] + 1, chunk); };
    for (;; chunk *= 2) {  // keep the number of parts bounded
      int64_t parts = 0;
      for (int r = 0; r < b->num_reqs; r++)
        if (b->extend_lens[r] == 1 && chunks_of(r) > 1) parts += chunks_of(r) * Hkv;
      if (parts <= limits.decode) break;
    }
    for (int r = 0; r < b->num_reqs; r++) {
      if (b->extend_lens[r] != 1) continue;
      const int64_t L = (int64_t)b->prefix_lens[r] + 1, nc = chunks_of(r);
      for (int32_t h = 0; h < Hkv; h++) {
        if (nc > 1)
          plan.dec_merges.push_back(
              kvx::DecodeMerge{(int32_t)qo[(size_t)r], h, (int32_t)plan.dec_parts, (int32_t)nc});
        for (int64_t c = 0; c < nc; c++) {
          AttnUnit u;
          u.qo_row0 = (int32_t)qo[(size_t)r];
          u.q_pos0 = b->prefix_lens[r];
          u.page_base = b->page_indptr[r];
          u.key_begin = (int32_t)(c * chunk);
          u.key_end = (int32_t)std::min<int64_t>(L, (c + 1) * chunk);
          u.head_ntok = (h << 16) | kvx::kDecodeUnitFlag | 1;
          u.part = nc > 1 ? (int32_t)plan.dec_parts++ : -1;
          u.req = r;
          dec_units.push_back(u);
        }
      }
    }
    std::stable_sort(dec_units.begin(), dec_units.end(), [](const AttnUnit& x, const AttnUnit& y) {
      return x.key_end - x.key_begin > y.key_end - y.key_begin;
    });
    filler.units = ceil_div((int64_t)dec_units.size(), Hkv);
    filler.cost = (double)(one_keys / BN) / (double)dec_units.size() * kDecodePerIter + kUnitCosts128.start;
  }

  int64_t split = split_keys > 0 || packed ? split_keys : choose_split(tiles, Hkv, tile_tok, D, filler, limits.prefill);
  auto boundaries = [&](const Tile& t) { return split > 0 ? t.qpos0 / split : 0; };  // split, 2 split, ... <= qpos0
  while (split > 0) {  // keep the number of parts bounded
    int64_t parts = 0;
    for (const Tile& t : tiles)
      if (const int64_t nb = boundaries(t)) parts += nb + 1;
    if (parts * Hkv <= limits.prefill) break;
    split *= 2;
  }

  // XCD of a unit.  Multiples of 8 heads: head h -> XCD h % 8.  Otherwise greedy by cost,
  // costliest first, each to the least loaded XCD: the tiles over one (request, head,
  // part), in runs of at most a sixth of an XCD's share of the work (13 requests of 2
  // heads, a request and head together: the busiest XCD 1.45 times the mean).
  const bool by_head = Hkv % kvx::kNumXcd == 0;
  std::vector<int32_t> run_of(tiles.size(), 0);  // the tile's run within its request
  if (!by_head) {
    int64_t total = 0, in_run = 0;
    for (const Tile& t : tiles) total += ceil_div(t.kend, BN);
    // an unsplit batch of less than four rounds: every tile by itself, since a tile
    // more or less is a third of a round there
    const int64_t most =
        split == 0 && (int64_t)tiles.size() * Hkv < 4 * kPlanSlots ? 0 : total * Hkv / (6 * kvx::kNumXcd);
    for (size_t k = 0; k < tiles.size(); k++) {
      const int64_t c = ceil_div(boundaries(tiles[k]) > 0 ? split : tiles[k].kend, BN);
      const bool same = k > 0 && tiles[k].r == tiles[k - 1].r;
      const bool fits = same && in_run + c <= most;
      run_of[k] = !same ? 0 : run_of[k - 1] + (fits ? 0 : 1);
      in_run = fits ? in_run + c : c;
    }
  }
  std::vector<size_t> bind_at((size_t)b->num_reqs, 0);  // first entry of a request: [head][run][part]
  std::vector<int32_t> bind_parts((size_t)b->num_reqs, 0), bind_n((size_t)b->num_reqs, 0);  // parts; runs x parts
  std::vector<uint8_t> bind_xcd;
  if (!by_head) {
    std::vector<int64_t> cost;
    for (size_t first = 0; first < tiles.size();) {
      size_t last = first;
      while (last < tiles.size() && tiles[last].r == tiles[first].r) last++;
      const size_t r = (size_t)tiles[first].r;
      // the request's longest tile has the most parts, its last tile is in the last run
      bind_at[r] = cost.size();
      bind_parts[r] = (int32_t)boundaries(tiles[first]) + 1;
      bind_n[r] = (run_of[last - 1] + 1) * bind_parts[r];
      cost.resize(cost.size() + (size_t)bind_n[r] * Hkv, 0);
      for (size_t k = first; k < last; k++) {
        const int64_t nb = boundaries(tiles[k]);
        for (int64_t i = 0; i <= nb; i++)
          for (int32_t h = 0; h < Hkv; h++)
            cost[bind_at[r] + (size_t)h * bind_n[r] + (size_t)(run_of[k] * bind_parts[r] + i)] +=
                ceil_div((i < nb ? (i + 1) * split : tiles[k].kend) - i * split, BN);
      }
      first = last;
    }
    std::vector<int32_t> by_cost(cost.size());
    std::iota(by_cost.begin(), by_cost.end(), 0);
    std::stable_sort(by_cost.begin(), by_cost.end(),
                     [&](int32_t x, int32_t y) { return cost[(size_t)x] > cost[(size_t)y]; });
    bind_xcd.resize(cost.size());
    int64_t load[kvx::kNumXcd] = {0};
    for (const int32_t i : by_cost) {
      int best = 0;
      for (int x = 1; x < kvx::kNumXcd; x++)
        if (load[x] < load[best]) best = x;
      bind_xcd[(size_t)i] = (uint8_t)best;
      load[best] += cost[(size_t)i];
    }
  }

  struct Placed {
    AttnUnit u;
    int32_t tok0;
    uint32_t code;
  };
  plan.tiles.clear();
  plan.codes.clear();
  plan.split = split;
  const bool coded = !plan.mixed && tiles.size() < kvx::kPlanTiles - 1 && tiles.size() * 6 < (size_t)kvx::kPlanWords &&
                     (uint32_t)Hkv <= kvx::kPlanHeads;
  std::vector<Placed> per_xcd[kvx::kNumXcd];
  plan.merges.clear();
  plan.n_parts = 0;
  int64_t most_ranges = 0;
  for (size_t first = 0; first < tiles.size();) {  // one request at a time
    size_t last = first;
    while (last < tiles.size() && tiles[last].r == tiles[first].r) last++;
    const int32_t r = tiles[first].r;
    // part numbers: a tile's parts are consecutive for each KV head
    std::vector<int64_t> part0;
    for (size_t k = first; k < last; k++) {
      const Tile& t = tiles[k];
      const int64_t nb = boundaries(t);
      part0.push_back(plan.n_parts);
      if (coded)
        plan.tiles.push_back(kvx::PlanTile{(int32_t)(qo[(size_t)r] + t.tok0), (int32_t)t.qpos0, b->page_indptr[r],
                                           (int32_t)t.kend, t.ntok << 16 | (int32_t)std::min<int64_t>(nb, 0xFFFF),
                                           (int32_t)plan.n_parts});
      if (nb == 0) continue;
      for (int32_t h = 0; h < Hkv; h++)
        plan.merges.push_back(MergeUnit{(int32_t)(qo[(size_t)r] + t.tok0), (h << 16) | t.ntok,
                                        (int32_t)(plan.n_parts + h * (nb + 1)), (int32_t)nb + 1});
      plan.n_parts += (nb + 1) * Hkv;
    }
    const int64_t ranges = boundaries(tiles[first]) + 1;
    most_ranges = std::max(most_ranges, ranges);
    for (int64_t i = 0; i < ranges; i++) {
      for (size_t k = first; k < last; k++) {
        const Tile& t = tiles[k];
        const int64_t nb = boundaries(t);
        if (i > nb) continue;
        AttnUnit u;
        u.qo_row0 = (int32_t)(qo[(size_t)r] + t.tok0);
        u.q_pos0 = (int32_t)t.qpos0;
        u.page_base = b->page_indptr[r];
        u.key_begin = (int32_t)(i * split);
        u.key_end = (int32_t)(i < nb ? (i + 1) * split : t.kend);
        u.req = r;
        for (int32_t h = 0; h < Hkv; h++) {
          const int x = by_head ? h % kvx::kNumXcd
                                : bind_xcd[bind_at[(size_t)r] + (size_t)h * bind_n[(size_t)r] +
                                           (size_t)(run_of[k] * bind_parts[(size_t)r] + i)];
          u.head_ntok = (h << 16) | t.ntok;
          u.part = nb > 0 ? (int32_t)(part0[k - first] + h * (nb + 1) + i) : -1;
          per_xcd[x].push_back(Placed{u, t.tok0, kvx::plan_code((uint32_t)k, (uint32_t)h, (uint32_t)i)});
        }
      }
    }
    first = last;
  }
  if (plan.n_parts > 0 || (int64_t)tiles.size() * Hkv < 4 * kPlanSlots)
    for (auto& v : per_xcd)
      std::stable_sort(v.begin(), v.end(), [](const Placed& x, const Placed& y) {
        return x.u.key_end - x.u.key_begin > y.u.key_end - y.u.key_begin;
      });
  if (plan.mixed) {
    for (int x = 0; x < kvx::kNumXcd; x++) {
      std::vector<Placed>& pre = per_xcd[x];
      std::vector<Placed> dec, all;
      for (size_t i = (size_t)x; i < dec_units.size(); i += kvx::kNumXcd) dec.push_back(Placed{dec_units[i], 0, 0});
      // An XCD's units go to its four shader engines strictly in turn (unit k to engine
      // k % 4, 8 CUs each) and in order, so that every engine must get both kinds alike:
      // they alternate in groups of four.
      constexpr size_t SE = 4;
      double total = 0.0, done = 0.0;
      for (const Placed& e : pre) total += (double)(e.u.key_end - e.u.key_begin);
      size_t next = 0;
      for (size_t i = 0; i < pre.size(); i++) {
        all.push_back(pre[i]);
        done += (double)(pre[i].u.key_end - pre[i].u.key_begin);
        if (i % SE != SE - 1) continue;
        const size_t due = (size_t)(kDecodeSpread * (double)dec.size() * done / total) / SE * SE;
        while (next < due && next < dec.size()) all.push_back(dec[next++]);
      }
      while (next < dec.size()) all.push_back(dec[next++]);
      pre.swap(all);
    }
  }
  size_t longest = 0;
  for (const auto& v : per_xcd) longest = std::max(longest, v.size());
  plan.units.clear();
  plan.items.clear();
  plan.units.reserve(longest * kvx::kNumXcd);
  if (plan.inspect) plan.items.reserve(longest * kvx::kNumXcd);
  for (size_t i = 0; i < longest; i++) {
    for (int x = 0; x < kvx::kNumXcd; x++) {
      if (i < per_xcd[x].size()) {
        const AttnUnit& u = per_xcd[x][i].u;
        plan.units.push_back(u);
        if (coded) plan.codes.push_back(per_xcd[x][i].code);
        if (!plan.inspect) continue;
        const bool dec = (u.head_ntok & kvx::kDecodeUnitFlag) != 0;
        // inspected part numbers are dense: decode parts follow the prefill parts
        const int32_t part = dec && u.part >= 0 ? (int32_t)plan.n_parts + u.part : u.part;
        plan.items.push_back(kvx_work_item{u.req, u.head_ntok >> 16, per_xcd[x][i].tok0, u.head_ntok & 0x7FFF,
                                           u.key_begin, u.key_end, part, x});
      } else if (!packed) {
        AttnUnit pad{};
        pad.part = -1;
        plan.units.push_back(pad);
        if (coded) plan.codes.push_back(kvx::kPlanPad);
        if (plan.inspect) plan.items.push_back(kvx_work_item{-1, 0, 0, 0, 0, 0, -1, x});
      }
    }
  }
  // drop trailing padding
  while (!plan.units.empty() && plan.units.back().key_end <= plan.units.back().key_begin) {
    plan.units.pop_back();
    if (plan.inspect) plan.items.pop_back();
    if (coded) plan.codes.pop_back();
  }
  if (most_ranges > (int64_t)kvx::kPlanRanges) plan.codes.clear();
  return KVX_OK;
}

// ---- decode steps: every request with work has exactly one suffix token
using kvx::DecodeMerge;
using kvx::DecodeUnit;

struct DecodePlan {
  std::vector<DecodeUnit> units;
  std::vector<DecodeMerge> merges;
  bool inspect = false;  // as in Plan
  std::vector<kvx_work_item> items;
  int64_t n_parts = 0;
};

bool is_decode_batch(const kvx_batch* b, int32_t Hq, int32_t Hkv) {
  if (Hq / Hkv > kvx::kDecodeMaxGroup) return false;
  bool any = false;
  for (int r = 0; r < b->num_reqs; r++) {
    if (b->extend_lens[r] > 1) return false;
    any |= b->extend_lens[r] == 1;
  }
  return any;
}

// Work plan of a decode step: each (request, KV head) key range [0, P] is cut into
// chunks of a common length, a multiple of 64 keys chosen so that the batch yields
// about 2048 chunks (8 per CU, of which two to four run at a time), at
// least 512 keys each; a range of more than one chunk becomes parts merged by
// log-sum-exp.  Chunks are dispatched longest first.
int make_decode_plan(const kvx_batch* b, const std::vector<int64_t>& qo, int32_t Hkv, int32_t split_keys,
                     int64_t max_parts, DecodePlan& plan) {
  const int64_t A = kvx::kDecodeChunkAlign;
  int64_t total = 0;
  for (int r = 0; r < b->num_reqs; r++)
    if (b->extend_lens[r] == 1) total += (int64_t)Hkv * ((int64_t)b->prefix_lens[r] + 1);
  int64_t chunk;
  if (split_keys > 0) {
    chunk = split_keys;
  } else {
    chunk = std::max<int64_t>(512, (total + 2047) / 2048);
    chunk = (chunk + A - 1) / A * A;
  }
  for (;;) {  // bound the partial results like the prefill planner does
    int64_t parts = 0;
    for (int r = 0; r < b->num_reqs; r++) {
      if (b->extend_lens[r] != 1) continue;
      const int64_t n = ((int64_t)b->prefix_lens[r] + 1 + chunk - 1) / chunk;
      if (n > 1) parts += n * Hkv;
    }
    if (parts <= max_parts) break;
    chunk *= 2;
  }
  for (int r = 0; r < b->num_reqs; r++) {
    if (b->extend_lens[r] != 1) continue;
    const int64_t L = (int64_t)b->prefix_lens[r] + 1;
    const int64_t nc = (L + chunk - 1) / chunk;
    const int64_t part0 = plan.n_parts;
    for (int64_t c = 0; c < nc; c++) {
      for (int32_t h = 0; h < Hkv; h++) {  // heads side by side (see InlinePlan)
        DecodeUnit u{};
        u.qo_row = (int32_t)qo[(size_t)r];
        u.page_base = b->page_indptr[r];
        u.key_begin = (int32_t)(c * chunk);
        u.key_end = (int32_t)std::min<int64_t>(L, (c + 1) * chunk);
        u.head = h;
        u.part = nc > 1 ? (int32_t)(part0 + h * nc + c) : -1;
        u.req = r;
        plan.units.push_back(u);
      }
    }
    if (nc > 1) {
      for (int32_t h = 0; h < Hkv; h++)
        plan.merges.push_back(DecodeMerge{(int32_t)qo[(size_t)r], h, (int32_t)(part0 + h * nc), (int32_t)nc});
      plan.n_parts += nc * Hkv;
    }
  }
  std::stable_sort(plan.units.begin(), plan.units.end(), [](const DecodeUnit& x, const DecodeUnit& y) {
    return x.key_end - x.key_begin > y.key_end - y.key_begin;
  });
  for (size_t i = 0; plan.inspect && i < plan.units.size(); i++) {
    const DecodeUnit& u = plan.units[i];
    kvx_work_item it{u.req, u.head, 0, 1, u.key_begin, u.key_end, u.part, (int32_t)(i % kvx::kNumXcd)};
    plan.items.push_back(it);
  }
  return KVX_OK;
}

int check_heads(int32_t Hq, int32_t Hkv, int32_t D) {
  if (Hkv <= 0 || Hq <= 0 || Hq % Hkv != 0)
    return fail(KVX_EINVAL, "num_q_heads (%d) must be a positive multiple of num_kv_heads (%d)", Hq, Hkv);
  if (Hq / Hkv > kvx::kTileRows)
    return fail(KVX_EUNSUPPORTED, "query heads per KV head (%d) above %d", Hq / Hkv, kvx::kTileRows);
  if (Hkv >= (1 << 15)) return fail(KVX_EUNSUPPORTED, "num_kv_heads too large");
  if (D != 64 && D != 128) return fail(KVX_EUNSUPPORTED, "head_dim %d (supported: 64, 128)", D);
  return KVX_OK;
}

// Where one attention call keeps its plan and its partial results: the pool's
// growable buffers, or the caller-independent fixed scratch of the allocation-free
// entry point (plan region, then partial-result region).
struct CallBuffers {
  kvx_pool* pool;
  const kvx::FixedScratch* fixed;
  uint8_t* base = nullptr;  // fixed scratch on the pool's device (after bind())

  // Bound on split parts of `per_part` bytes each.
  int64_t max_parts(size_t per_part) const {
    if (!fixed) return kMaxParts;
    return std::min<int64_t>(kMaxParts, (int64_t)(fixed->parts_bytes / per_part));
  }
  // Host-only size check of the plan (before any device call).
  int check_plan(size_t bytes) const {
    if (fixed && bytes > fixed->plan_bytes)
      return fail(KVX_EUNSUPPORTED, "work plan of %zu bytes exceeds the fixed scratch's %zu-byte plan region",
                  bytes, fixed->plan_bytes);
    return KVX_OK;
  }
  // With the pool's device current: the fixed scratch's address on it.
  int bind() {
    if (!fixed) return KVX_OK;
    void* p = nullptr;
    if (int rc = fixed->address(pool->device, &p)) return rc;
    base = (uint8_t*)p;
    return KVX_OK;
  }
  int parts(size_t bytes, hipStream_t s, float** out) {
    if (fixed) {
      if (bytes > fixed->parts_bytes)
        return fail(KVX_EUNSUPPORTED, "partial results of %zu bytes exceed the fixed scratch's %zu bytes", bytes,
                    fixed->parts_bytes);
      *out = (float*)(base + fixed->plan_bytes);
      return KVX_OK;
    }
    if (int rc = pool->parts.ensure(bytes, s)) return rc;
    *out = (float*)pool->parts.ptr;
    return KVX_OK;
  }
  int upload(const std::vector<uint8_t>& blob, hipStream_t s, void** out) {
    if (fixed) {
      // pageable source: the copy is staged before the call returns
      KVX_HIP(hipMemcpyAsync(base, blob.data(), blob.size(), hipMemcpyHostToDevice, s));
      *out = base;
      return KVX_OK;
    }
    return pool->st_attn.upload(blob.data(), blob.size(), s, out);
  }
  // staged: the call's kernels read the staging buffer
  int done(hipStream_t s, bool staged) {
    if (fixed) return KVX_OK;
    if (staged)
      if (int rc = pool->st_attn.done(s)) return rc;
    return pool->parts.done(s);
  }
};

// The units of a decode plan in kernel arguments, if they fit (see InlinePlan).
bool inline_units(const std::vector<DecodeUnit>& units, kvx::InlinePlan<DecodeUnit>& out) {
  constexpr int32_t H = kvx::kNumXcd;
  out.n = 0;
  if (units.size() > (size_t)kvx::kInlineUnits * H) return false;
  bool grouped = units.size() % H == 0;
  for (size_t i = 0; grouped && i < units.size(); i += H) {
    const int32_t part = units[i].part, stride = part < 0 ? 0 : units[i + 1].part - part;
    for (int32_t h = 1; grouped && h < H; h++) {
      DecodeUnit x = units[i];
      x.head += h;
      x.part = part < 0 ? -1 : part + h * stride;
      grouped = std::memcmp(&x, &units[i + (size_t)h], sizeof x) == 0;
    }
  }
  if (!grouped && units.size() > (size_t)kvx::kInlineUnits) return false;
  out.heads = grouped ? H : 1;
  for (size_t i = 0; i < units.size(); i += (size_t)out.heads) {
    DecodeUnit e = units[i];
    e.req = grouped && e.part >= 0 ? units[i + 1].part - e.part : 0;
    out.unit[out.n++] = e;
  }
  return true;
}

// A prefill plan in kernel arguments, if it fits (see CompactPlan).
bool compact_plan(const Plan& plan, kvx::CompactPlan& out) {
  constexpr int32_t H = kvx::kNumXcd;
  const std::vector<uint32_t>& c = plan.codes;
  const size_t room = (size_t)kvx::kPlanWords - std::min<size_t>(kvx::kPlanWords, 6 * plan.tiles.size());
  if (c.empty() || c.size() > room * H) return false;
  bool grouped = c.size() % H == 0;
  for (size_t i = 0; grouped && i < c.size(); i++)
    grouped = c[i] != kvx::kPlanPad && c[i] == c[i / H * H] + kvx::plan_code(0, (uint32_t)(i % H), 0);
  if (!grouped && c.size() > room) return false;
  out.n = (int32_t)c.size();
  out.n_tiles = (int32_t)plan.tiles.size();
  out.heads = grouped ? H : 1;
  out.split = (int32_t)plan.split;
  static_assert(sizeof(kvx::PlanTile) == 6 * sizeof(uint32_t), "six words per tile");
  std::memcpy(out.words, plan.tiles.data(), plan.tiles.size() * sizeof(kvx::PlanTile));
  uint32_t* w = out.words + 6 * plan.tiles.size();
  for (size_t i = 0; i < c.size(); i += (size_t)out.heads) *w++ = c[i];
  return true;
}

// The merges of either kind of plan in kernel arguments, if they fit; they go tile by tile
// (request by request) with all KV heads.
template <typename M>
bool inline_merges(const std::vector<M>& merges, int32_t Hkv, kvx::InlineMerges<M>& out) {
  out.n = 0;
  if (merges.size() > (size_t)kvx::kInlineMerges * Hkv) return false;
  out.heads = Hkv;
  for (size_t i = 0; i < merges.size(); i += (size_t)Hkv) out.merge[out.n++] = merges[i];
  return true;
}

template <typename U, typename M>
std::vector<uint8_t> plan_blob(const std::vector<U>& units, const std::vector<M>& merges,
                               const std::vector<DecodeMerge>& dec_merges = {}) {
  const size_t ub = units.size() * sizeof(U), mb = merges.size() * sizeof(M), db = dec_merges.size() * sizeof(DecodeMerge);
  std::vector<uint8_t> blob(ub + mb + db);
  if (ub) std::memcpy(blob.data(), units.data(), ub);
  if (mb) std::memcpy(blob.data() + ub, merges.data(), mb);
  if (db) std::memcpy(blob.data() + ub + mb, dec_merges.data(), db);
  return blob;
}

// The requests of a store batch in the kernel arguments when there are few enough
// (returns false otherwise: the unit list is uploaded instead).  Workgroup order
// matches the unit lists below: request by request, logical page by page.
bool inline_store_reqs(const kvx_batch* b, const std::vector<int64_t>& qo, kvx::StoreReqs& rq) {
  rq.n = 0;
  int32_t wg = 0;
  for (int r = 0; r < b->num_reqs; r++) {
    const int64_t P = b->prefix_lens[r], E = b->extend_lens[r];
    if (E == 0) continue;
    if (rq.n == kvx::kStoreInlineReqs) {
      rq.n = 0;
      return false;
    }
    const int64_t pages = (P + E - 1) / kvx::kPageSize - P / kvx::kPageSize + 1;
    rq.first[rq.n] = wg;
    rq.qo[rq.n] = (int32_t)qo[(size_t)r];
    rq.prefix[rq.n] = (int32_t)P;
    rq.end[rq.n] = (int32_t)(P + E);
    rq.page_base[rq.n] = b->page_indptr[r];
    wg += (int32_t)pages;
    rq.n++;
  }
  rq.first[rq.n] = wg;
  return rq.n > 0;
}

// A decode batch that reads more K/V than the 256 MB Infinity Cache holds may use non-temporal
// loads (see decode_kernel).  Smaller batches find pages there that were just stored or read
// (48 MB: 30.4 us, 31.8 us non-temporal), and in one of more than kShareReqs requests the look at
// every page list would cost each unit more than these loads give.
constexpr int64_t kStreamBytes = 256ll << 20;

int decode_attention(kvx_pool* pool, const kvx_batch* batch, const std::vector<int64_t>& qo, const void* q,
                     int32_t num_q_heads, float sm_scale, void* out, float* lse, hipStream_t s, CallBuffers& buf) {
  const int D = pool->head_dim;
  constexpr int R = kvx::kDecodeMaxGroup;
  DecodePlan plan;
  if (int rc = make_decode_plan(batch, qo, pool->num_kv_heads, pool->split_keys,
                                buf.max_parts((size_t)R * (D + 1) * sizeof(float)), plan))
    return rc;
  kvx::DecodeParams dp;
  kvx::DecodeMergeParams m;
  const bool in_args = inline_merges(plan.merges, pool->num_kv_heads, m.plan) && inline_units(plan.units, dp.plan);
  std::vector<uint8_t> blob;
  if (!in_args) {
    dp.plan.n = m.plan.n = 0;
    blob = plan_blob(plan.units, plan.merges);
  }
  int64_t kv_bytes = 0;  // K and V, page lists that share pages counted each
  std::vector<int32_t> lists;
  for (int r = 0; r < batch->num_reqs; r++) {
    if (batch->extend_lens[r] != 1) continue;
    kv_bytes += 2 * ((int64_t)batch->prefix_lens[r] + 1) * pool->num_kv_heads * D * pool->elem_bytes;
    lists.push_back(batch->page_indptr[r]);
  }
  const bool streams = kv_bytes > kStreamBytes && lists.size() <= (size_t)kvx::kShareReqs;
  dp.lists.base = nullptr;
  dp.lists.n = streams ? (int32_t)lists.size() : 0;
  const size_t lists_at = blob.size();
  if (streams) {
    lists.push_back(batch->page_indptr[batch->num_reqs]);
    const size_t bytes = lists.size() * sizeof(int32_t);
    if (in_args) {
      std::memcpy(dp.lists.in_args, lists.data(), bytes);  // every request has an entry of its own
    } else if (!buf.fixed || lists_at + bytes <= buf.fixed->plan_bytes) {
      blob.resize(lists_at + bytes);
      std::memcpy(blob.data() + lists_at, lists.data(), bytes);
    } else {
      dp.lists.n = 0;
    }
  }
  if (int rc = buf.check_plan(blob.size())) return rc;
  if (int rc = use_device(pool)) return rc;
  if (validate_mode())
    if (int rc = check_page_ids(pool, batch, s)) return rc;
  if (int rc = buf.bind()) return rc;
  float* parts = nullptr;
  if (plan.n_parts > 0)
    if (int rc = buf.parts((size_t)plan.n_parts * R * (D + 1) * sizeof(float), s, &parts)) return rc;
  void* dev = nullptr;
  if (!in_args)
    if (int rc = buf.upload(blob, s, &dev)) return rc;
  kvx::DecodeArgs& p = dp.a;
  p.q = (const uint16_t*)q;
  p.out = (uint16_t*)out;
  p.lse = lse;
  p.k_pool = pool->k;
  p.v_pool = pool->v;
  p.page_ids = batch->page_ids;
  dp.units = (const DecodeUnit*)dev;
  p.o_part = plan.n_parts ? parts : nullptr;
  p.lse_part = plan.n_parts ? parts + (size_t)plan.n_parts * R * D : nullptr;
  p.k_scale = pool->scales_d;
  p.v_scale = pool->scales_d ? pool->scales_d + pool->num_kv_heads : nullptr;
  p.num_q_heads = num_q_heads;
  p.num_kv_heads = pool->num_kv_heads;
  p.group = num_q_heads / pool->num_kv_heads;
  p.scale_log2 = sm_scale * 1.4426950408889634f;
  if (!in_args && dp.lists.n > 0) dp.lists.base = (const int32_t*)((const uint8_t*)dev + lists_at);
  hipError_t e = kvx::launch_decode(dp, (int64_t)plan.units.size(), D, pool->kv_dtype == KVX_KV_FP8_E4M3, s);
  if (e != hipSuccess) return hip_fail(e, "decode kernel launch");
  if (!plan.merges.empty()) {
    m.merges = (const DecodeMerge*)((const uint8_t*)dev + plan.units.size() * sizeof(DecodeUnit));
    m.o_part = p.o_part;
    m.lse_part = p.lse_part;
    m.out = (uint16_t*)out;
    m.lse = lse;
    m.num_q_heads = num_q_heads;
    m.group = p.group;
    e = kvx::launch_decode_merge(m, (int64_t)plan.merges.size(), D, s);
    if (e != hipSuccess) return hip_fail(e, "decode merge kernel launch");
  }
  return buf.done(s, !in_args);
}

}  // namespace

extern "C" {

const char* kvx_last_error(void) { return g_last_error.c_str(); }

int kv_pool_set_split_keys(kvx_pool* pool, int32_t keys) {
  g_last_error.clear();
  if (int rc = check_pool(pool)) return rc;
  if (keys < 0 || keys % kvx::kTileKeys != 0)
    return fail(KVX_EINVAL, "split keys %d: must be 0 or a positive multiple of %d", keys, kvx::kTileKeys);
  pool->split_keys = keys;
  return KVX_OK;
}

int kv_pool_set_scaled_q(kvx_pool* pool, int32_t enable) {
  g_last_error.clear();
  if (int rc = check_pool(pool)) return rc;
  if (enable != 0 && enable != 1) return fail(KVX_EINVAL, "scaled_q %d: must be 0 or 1", enable);
  pool->scaled_q = enable;
  return KVX_OK;
}

int kv_pool_create(int64_t num_pages, int32_t page_size, int32_t num_kv_heads, int32_t head_dim,
                   int32_t kv_dtype, const float* k_scale, const float* v_scale, kvx_pool** out) {
  g_last_error.clear();
  if (out == nullptr) return fail(KVX_EINVAL, "out is NULL");
  *out = nullptr;
  if (num_pages <= 0) return fail(KVX_EINVAL, "num_pages = %lld must be > 0", (long long)num_pages);
  if (num_pages > (int64_t)INT32_MAX) return fail(KVX_EINVAL, "num_pages above 2^31-1");
  if (num_kv_heads <= 0) return fail(KVX_EINVAL, "num_kv_heads = %d must be > 0", num_kv_heads);
  if (num_kv_heads >= (1 << 15)) return fail(KVX_EUNSUPPORTED, "num_kv_heads too large");
  if (page_size != kvx::kPageSize) return fail(KVX_EUNSUPPORTED, "page_size %d (supported: 16)", page_size);
  if (head_dim != 64 && head_dim != 128) return fail(KVX_EUNSUPPORTED, "head_dim %d (supported: 64, 128)", head_dim);
  if (kv_dtype != KVX_KV_BF16 && kv_dtype != KVX_KV_FP8_E4M3) return fail(KVX_EINVAL, "kv_dtype %d", kv_dtype);
  if (kv_dtype == KVX_KV_FP8_E4M3) {
    if (!k_scale || !v_scale) return fail(KVX_EUNSUPPORTED, "an fp8 pool needs k_scale and v_scale");
    for (int h = 0; h < num_kv_heads; h++)
      if (!(std::isfinite(k_scale[h]) && k_scale[h] > 0.f && std::isfinite(v_scale[h]) && v_scale[h] > 0.f))
        return fail(KVX_EINVAL, "fp8 scales of head %d must be finite and > 0", h);
  }
  const int eb = kv_dtype == KVX_KV_BF16 ? 2 : 1;
  const size_t bytes = (size_t)num_pages * num_kv_heads * page_size * head_dim * eb;
  if (bytes / (size_t)num_pages / (size_t)eb != (size_t)num_kv_heads * page_size * head_dim)
    return fail(KVX_EINVAL, "pool size overflows");
  kvx_pool* p = new kvx_pool();
  p->num_pages = num_pages;
  p->page_size = page_size;
  p->num_kv_heads = num_kv_heads;
  p->head_dim = head_dim;
  p->kv_dtype = kv_dtype;
  p->elem_bytes = eb;
  auto cleanup = [&](int rc) {
    if (p->k) (void)hipFree(p->k);
    if (p->v) (void)hipFree(p->v);
    if (p->scales_d) (void)hipFree(p->scales_d);
    delete p;
    return rc;
  };
  hipError_t e = hipGetDevice(&p->device);
  if (e != hipSuccess) return cleanup(hip_fail(e, "hipGetDevice"));
  e = hipMalloc(&p->k, bytes);
  if (e != hipSuccess) return cleanup(hip_fail(e, "hipMalloc(K pool)"));
  e = hipMalloc(&p->v, bytes);
  if (e != hipSuccess) return cleanup(hip_fail(e, "hipMalloc(V pool)"));
  e = hipMemset(p->k, 0, bytes);
  if (e == hipSuccess) e = hipMemset(p->v, 0, bytes);
  if (e != hipSuccess) return cleanup(hip_fail(e, "hipMemset(pool)"));
  if (kv_dtype == KVX_KV_FP8_E4M3) {
    std::vector<float> s((size_t)4 * num_kv_heads);
    for (int h = 0; h < num_kv_heads; h++) {
      s[(size_t)h] = k_scale[h];
      s[(size_t)num_kv_heads + h] = v_scale[h];
      s[(size_t)2 * num_kv_heads + h] = 1.0f / k_scale[h];  // fp32 reciprocal used to quantise
      s[(size_t)3 * num_kv_heads + h] = 1.0f / v_scale[h];
    }
    e = hipMalloc(&p->scales_d, s.size() * sizeof(float));
    if (e == hipSuccess) e = hipMemcpy(p->scales_d, s.data(), s.size() * sizeof(float), hipMemcpyHostToDevice);
    if (e != hipSuccess) return cleanup(hip_fail(e, "fp8 scales"));
  }
  e = hipDeviceSynchronize();
  if (e != hipSuccess) return cleanup(hip_fail(e, "hipDeviceSynchronize"));
  *out = p;
  return KVX_OK;
}

int kv_pool_destroy(kvx_pool* pool) {
  g_last_error.clear();
  if (pool == nullptr) return KVX_OK;
  (void)use_device(pool);
  hipError_t e = hipDeviceSynchronize();
  pool->st_store.release();
  pool->st_attn.release();
  pool->st_io.release();
  pool->st_move.release();
  pool->parts.release();
  if (pool->k) (void)hipFree(pool->k);
  if (pool->v) (void)hipFree(pool->v);
  if (pool->scales_d) (void)hipFree(pool->scales_d);
  delete pool;
  if (e != hipSuccess) return hip_fail(e, "hipDeviceSynchronize");
  return KVX_OK;
}

int kv_pool_layout(const kvx_pool* pool, kvx_pool_layout* out) {
  g_last_error.clear();
  if (int rc = check_pool(pool)) return rc;
  if (out == nullptr) return fail(KVX_EINVAL, "out is NULL");
  const int64_t S = pool->page_size, D = pool->head_dim, H = pool->num_kv_heads;
  std::memset(out, 0, sizeof *out);
  out->k_base = pool->k;
  out->v_base = pool->v;
  out->num_pages = pool->num_pages;
  out->page_size = pool->page_size;
  out->num_kv_heads = pool->num_kv_heads;
  out->head_dim = pool->head_dim;
  out->kv_dtype = pool->kv_dtype;
  out->elem_bytes = pool->elem_bytes;
  out->k_stride_page = H * S * D;
  out->k_stride_head = S * D;
  out->k_stride_slot = D;
  out->k_stride_dim = 1;
  out->v_stride_page = H * S * D;
  out->v_stride_head = S * D;
  out->v_stride_slot = 1;
  out->v_stride_dim = S;
  out->k_scale = pool->scales_d;
  out->v_scale = pool->scales_d ? pool->scales_d + H : nullptr;
  return KVX_OK;
}

static int page_io(kvx_pool* pool, const int32_t* page_ids, int64_t n, void* k_lin, void* v_lin, int to_pool,
                   kvx_stream_t stream) {
  if (int rc = check_pool(pool)) return rc;
  if (n < 0) return fail(KVX_EINVAL, "n = %lld < 0", (long long)n);
  if (n == 0) return KVX_OK;
  if (!page_ids || !k_lin || !v_lin) return fail(KVX_EINVAL, "page_ids, K and V buffers must be non-NULL");
  if (int rc = check_align(k_lin, "K buffer")) return rc;
  if (int rc = check_align(v_lin, "V buffer")) return rc;
  if (n > (int64_t)INT32_MAX) return fail(KVX_EINVAL, "too many pages");
  for (int64_t i = 0; i < n; i++)
    if (page_ids[i] < 0 || page_ids[i] >= pool->num_pages)
      return fail(KVX_ERANGE, "page_ids[%lld] = %d outside [0, %lld)", (long long)i, page_ids[i],
                  (long long)pool->num_pages);
  if (int rc = use_device(pool)) return rc;
  hipStream_t s = (hipStream_t)stream;
  // Up to a few launches' worth of ids travel in kernel arguments instead of through a
  // copy and its wait (2000 pages out and in on new pools: 181 us with copies, 151 us without).
  const bool in_args = n <= 8 * kvx::kInlinePages;
  void* ids_d = nullptr;
  if (!in_args)
    if (int rc = pool->st_io.upload(page_ids, (size_t)n * sizeof(int32_t), s, &ids_d)) return rc;
  kvx::PageIoParams p;
  p.page_ids = (const int32_t*)ids_d;
  p.host_ids = in_args ? page_ids : nullptr;
  p.k_pool = pool->k;
  p.v_pool = pool->v;
  p.k_lin = k_lin;
  p.v_lin = v_lin;
  p.num_kv_heads = pool->num_kv_heads;
  p.to_pool = to_pool;
  hipError_t e = kvx::launch_page_io(p, n, pool->head_dim, pool->elem_bytes, s);
  if (e != hipSuccess) return hip_fail(e, "page io kernel launch");
  return in_args ? KVX_OK : pool->st_io.done(s);
}

int kv_pool_write_pages(kvx_pool* pool, const int32_t* page_ids, int64_t n, const void* k_src, const void* v_src,
                        kvx_stream_t stream) {
  g_last_error.clear();
  return page_io(pool, page_ids, n, const_cast<void*>(k_src), const_cast<void*>(v_src), 1, stream);
}

int kv_pool_read_pages(const kvx_pool* pool, const int32_t* page_ids, int64_t n, void* k_dst, void* v_dst,
                       kvx_stream_t stream) {
  g_last_error.clear();
  return page_io(const_cast<kvx_pool*>(pool), page_ids, n, k_dst, v_dst, 0, stream);
}

static int64_t record_bytes(const kvx_pool* pool) {
  return 2 * (int64_t)pool->num_kv_heads * kvx::kPageSize * pool->head_dim * pool->elem_bytes;
}

int kv_pool_record_bytes(const kvx_pool* pool, int64_t* bytes) {
  g_last_error.clear();
  if (int rc = check_pool(pool)) return rc;
  if (bytes == nullptr) return fail(KVX_EINVAL, "bytes is NULL");
  *bytes = record_bytes(pool);
  return KVX_OK;
}

// Spill (to_host) or reload whole pages between the pool and pinned host records.
static int page_move(kvx_pool* pool, const int32_t* page_ids, const int32_t* slots, int64_t n, const void* host,
                     int64_t host_slots, int to_host, kvx_stream_t stream) {
  if (int rc = check_pool(pool)) return rc;
  if (n < 0 || host_slots < 0) return fail(KVX_EINVAL, "n = %lld and host_slots = %lld must be >= 0", (long long)n,
                                           (long long)host_slots);
  if (n == 0) return KVX_OK;
  if (!page_ids || !slots || !host) return fail(KVX_EINVAL, "page_ids, slots and host must be non-NULL");
  if (int rc = check_align(host, "host")) return rc;
  if (n > (int64_t)INT32_MAX) return fail(KVX_EINVAL, "too many pages");
  for (int64_t i = 0; i < n; i++) {
    if (page_ids[i] < 0 || page_ids[i] >= pool->num_pages)
      return fail(KVX_ERANGE, "page_ids[%lld] = %d outside [0, %lld)", (long long)i, page_ids[i],
                  (long long)pool->num_pages);
    if (slots[i] < 0 || slots[i] >= host_slots)
      return fail(KVX_ERANGE, "slots[%lld] = %d outside [0, %lld)", (long long)i, slots[i], (long long)host_slots);
  }
  // the written side must not repeat: slots of a spill, pages of a reload
  std::vector<int32_t> dst(to_host ? slots : page_ids, (to_host ? slots : page_ids) + n);
  std::sort(dst.begin(), dst.end());
  if (std::adjacent_find(dst.begin(), dst.end()) != dst.end())
    return fail(KVX_EINVAL, "%s repeats an entry", to_host ? "slots" : "page_ids");
  if (int rc = use_device(pool)) return rc;
  hipPointerAttribute_t attr{};
  if (hipPointerGetAttributes(&attr, host) != hipSuccess || attr.type != hipMemoryTypeHost ||
      attr.devicePointer == nullptr) {
    (void)hipGetLastError();
    return fail(KVX_EINVAL, "host must be pinned host memory (hipHostMalloc, or a pinned torch tensor)");
  }
  const int64_t off = (const uint8_t*)host - (const uint8_t*)attr.hostPointer;
  hipStream_t s = (hipStream_t)stream;
  std::vector<int32_t> idx((size_t)(2 * n));
  std::copy(page_ids, page_ids + n, idx.begin());
  std::copy(slots, slots + n, idx.begin() + n);
  void* idx_d = nullptr;
  if (int rc = pool->st_move.upload(idx.data(), idx.size() * sizeof(int32_t), s, &idx_d)) return rc;
  kvx::PageMoveParams p;
  p.page_ids = (const int32_t*)idx_d;
  p.slots = (const int32_t*)idx_d + n;
  p.k_pool = (uint8_t*)pool->k;
  p.v_pool = (uint8_t*)pool->v;
  p.host = (uint8_t*)attr.devicePointer + (attr.hostPointer ? off : 0);
  p.block_bytes = record_bytes(pool) / 2;
  p.to_host = to_host;
  hipError_t e = kvx::launch_page_move(p, n, s);
  if (e != hipSuccess) return hip_fail(e, "page move kernel launch");
  return pool->st_move.done(s);
}

int kv_pool_spill(const kvx_pool* pool, const int32_t* page_ids, const int32_t* slots, int64_t n, void* host,
                  int64_t host_slots, kvx_stream_t stream) {
  g_last_error.clear();
  return page_move(const_cast<kvx_pool*>(pool), page_ids, slots, n, host, host_slots, 1, stream);
}

int kv_pool_reload(kvx_pool* pool, const int32_t* page_ids, const int32_t* slots, int64_t n, const void* host,
                   int64_t host_slots, kvx_stream_t stream) {
  g_last_error.clear();
  return page_move(pool, page_ids, slots, n, host, host_slots, 0, stream);
}

int store_kv(kvx_pool* pool, const kvx_batch* batch, const void* k_ext, const void* v_ext, kvx_stream_t stream) {
  g_last_error.clear();
  if (int rc = check_pool(pool)) return rc;
  std::vector<int64_t> qo;
  if (int rc = check_batch(batch, qo)) return rc;
  if (qo.back() == 0) return KVX_OK;
  if (!k_ext || !v_ext) return fail(KVX_EINVAL, "k_ext and v_ext must be non-NULL");
  if (int rc = check_align(k_ext, "k_ext")) return rc;
  if (int rc = check_align(v_ext, "v_ext")) return rc;
  if (int rc = use_device(pool)) return rc;
  hipStream_t s = (hipStream_t)stream;
  if (validate_mode())
    if (int rc = check_page_ids(pool, batch, s)) return rc;
  std::vector<StoreUnit> units;
  const int S = kvx::kPageSize;
  for (int r = 0; r < batch->num_reqs; r++) {
    const int64_t P = batch->prefix_lens[r], E = batch->extend_lens[r];
    if (E == 0) continue;
    const int64_t L = P + E;
    for (int64_t lp = P / S; lp <= (L - 1) / S; lp++) {
      StoreUnit u;
      u.row_slot0 = (int32_t)(qo[(size_t)r] + lp * S - P);
      u.page_pos = (int32_t)(batch->page_indptr[r] + lp);
      u.slot_begin = (int32_t)(std::max<int64_t>(P, lp * S) - lp * S);
      u.slot_end = (int32_t)(std::min<int64_t>(L, lp * S + S) - lp * S);
      units.push_back(u);
    }
  }
  kvx::StoreParams p;
  void* units_d = nullptr;
  if (!inline_store_reqs(batch, qo, p.reqs))
    if (int rc = pool->st_store.upload(units.data(), units.size() * sizeof(StoreUnit), s, &units_d)) return rc;
  p.k_ext = (const uint16_t*)k_ext;
  p.v_ext = (const uint16_t*)v_ext;
  p.k_pool = pool->k;
  p.v_pool = pool->v;
  p.page_ids = batch->page_ids;
  p.units = (const StoreUnit*)units_d;
  p.k_inv_scale = pool->scales_d ? pool->scales_d + 2 * pool->num_kv_heads : nullptr;
  p.v_inv_scale = pool->scales_d ? pool->scales_d + 3 * pool->num_kv_heads : nullptr;
  p.num_kv_heads = pool->num_kv_heads;
  hipError_t e = kvx::launch_store_kv(p, (int64_t)units.size(), pool->head_dim, pool->kv_dtype == KVX_KV_FP8_E4M3, s);
  if (e != hipSuccess) return hip_fail(e, "store_kv kernel launch");
  return p.reqs.n > 0 ? KVX_OK : pool->st_store.done(s);
}

int store_kv_rope(kvx_pool* pool, const kvx_batch* batch, const kvx_rope* rope, const void* q, int32_t num_q_heads,
                  void* q_out, const void* k_ext, const void* v_ext, kvx_stream_t stream) {
  g_last_error.clear();
  if (int rc = check_pool(pool)) return rc;
  std::vector<int64_t> qo;
  if (int rc = check_batch(batch, qo)) return rc;
  if (rope == nullptr) return fail(KVX_EINVAL, "rope is NULL");
  const int D = pool->head_dim;
  const int rd = rope->rotary_dim;
  if (rd < 16 || rd > D || rd % 16 != 0)
    return fail(KVX_EINVAL, "rotary_dim = %d must be a multiple of 16 in [16, head_dim = %d]", rd, D);
  if (rope->style != KVX_ROPE_HALF && rope->style != KVX_ROPE_INTERLEAVED)
    return fail(KVX_EINVAL, "style = %d", rope->style);
  if (!(rope->norm_eps >= 0.0f) || !std::isfinite(rope->norm_eps))
    return fail(KVX_EINVAL, "norm_eps must be finite and >= 0");
  kvx::RopeParams p{};
  for (int j = 0; j < rd / 2; j++) {
    double f;
    if (rope->inv_freq) {
      f = rope->inv_freq[j];
      if (!(f >= 0.0) || !std::isfinite(f)) return fail(KVX_EINVAL, "inv_freq[%d] must be finite and >= 0", j);
    } else {
      if (!(rope->theta > 0.0) || !std::isfinite(rope->theta))
        return fail(KVX_EINVAL, "theta must be finite and > 0");
      f = std::pow(rope->theta, -2.0 * j / rd);
    }
    p.rev_freq[j] = f / 6.283185307179586476925286766559;  // turns per position
  }
  if (num_q_heads < 0) return fail(KVX_EINVAL, "num_q_heads = %d < 0", num_q_heads);
  if (num_q_heads > 0 && (!q || !q_out)) return fail(KVX_EINVAL, "q and q_out must be non-NULL");
  if (num_q_heads > 0) {
    if (int rc = check_align(q, "q")) return rc;
    if (int rc = check_align(q_out, "q_out")) return rc;
  }
  if (int rc = check_align(rope->q_norm, "q_norm")) return rc;
  if (int rc = check_align(rope->k_norm, "k_norm")) return rc;
  if (qo.back() == 0) return KVX_OK;
  if (!k_ext || !v_ext) return fail(KVX_EINVAL, "k_ext and v_ext must be non-NULL");
  if (int rc = check_align(k_ext, "k_ext")) return rc;
  if (int rc = check_align(v_ext, "v_ext")) return rc;
  if (int rc = use_device(pool)) return rc;
  hipStream_t s = (hipStream_t)stream;
  if (validate_mode())
    if (int rc = check_page_ids(pool, batch, s)) return rc;
  std::vector<kvx::RopeUnit> units;
  const int S = kvx::kPageSize;
  for (int r = 0; r < batch->num_reqs; r++) {
    const int64_t P = batch->prefix_lens[r], E = batch->extend_lens[r];
    if (E == 0) continue;
    const int64_t L = P + E;
    for (int64_t lp = P / S; lp <= (L - 1) / S; lp++) {
      kvx::RopeUnit u;
      u.row_slot0 = (int32_t)(qo[(size_t)r] + lp * S - P);
      u.page_pos = (int32_t)(batch->page_indptr[r] + lp);
      u.slot_begin = (int32_t)(std::max<int64_t>(P, lp * S) - lp * S);
      u.slot_end = (int32_t)(std::min<int64_t>(L, lp * S + S) - lp * S);
      u.pos_slot0 = (int32_t)(lp * S);
      units.push_back(u);
    }
  }
  void* units_d = nullptr;
  if (!inline_store_reqs(batch, qo, p.reqs))
    if (int rc = pool->st_store.upload(units.data(), units.size() * sizeof(kvx::RopeUnit), s, &units_d)) return rc;
  p.q = (const uint16_t*)q;
  p.q_out = (uint16_t*)q_out;
  p.k_ext = (const uint16_t*)k_ext;
  p.v_ext = (const uint16_t*)v_ext;
  p.k_pool = pool->k;
  p.v_pool = pool->v;
  p.page_ids = batch->page_ids;
  p.units = (const kvx::RopeUnit*)units_d;
  p.k_inv_scale = pool->scales_d ? pool->scales_d + 2 * pool->num_kv_heads : nullptr;
  p.v_inv_scale = pool->scales_d ? pool->scales_d + 3 * pool->num_kv_heads : nullptr;
  p.q_norm = (const uint16_t*)rope->q_norm;
  p.k_norm = (const uint16_t*)rope->k_norm;
  p.num_q_heads = num_q_heads;
  p.num_kv_heads = pool->num_kv_heads;
  p.rotary_dim = rd;
  p.norm_eps = rope->norm_eps;
  hipError_t e = kvx::launch_store_kv_rope(p, (int64_t)units.size(), D, pool->kv_dtype == KVX_KV_FP8_E4M3,
                                           rope->style == KVX_ROPE_INTERLEAVED, s);
  if (e != hipSuccess) return hip_fail(e, "store_kv_rope kernel launch");
  return p.reqs.n > 0 ? KVX_OK : pool->st_store.done(s);
}

int extend_attention_plan(const kvx_batch* batch, int32_t num_q_heads, int32_t num_kv_heads, int32_t head_dim,
                          int32_t split_keys, kvx_work_item* items, int64_t cap, int64_t* count) {
  g_last_error.clear();
  if (count == nullptr) return fail(KVX_EINVAL, "count is NULL");
  *count = 0;
  if (int rc = check_heads(num_q_heads, num_kv_heads, head_dim)) return rc;
  if (split_keys < 0 || split_keys % kvx::kTileKeys != 0)
    return fail(KVX_EINVAL, "split keys %d: must be 0 or a positive multiple of %d", split_keys, kvx::kTileKeys);
  std::vector<int64_t> qo;
  if (int rc = check_batch(batch, qo, false)) return rc;
  if (cap < 0) return fail(KVX_EINVAL, "cap < 0");
  std::vector<kvx_work_item> out_items;
  if (qo.back() > 0) {
    if (is_decode_batch(batch, num_q_heads, num_kv_heads)) {
      DecodePlan dp;
      dp.inspect = true;
      if (int rc = make_decode_plan(batch, qo, num_kv_heads, split_keys, kMaxParts, dp)) return rc;
      out_items = std::move(dp.items);
    } else {
      Plan plan;
      plan.inspect = true;
      const bool mixed = is_mixed_batch(batch, num_q_heads, num_kv_heads);
      if (int rc = make_plan(batch, qo, num_q_heads, num_kv_heads, head_dim, split_keys, pool_limits(mixed), mixed, plan))
        return rc;
      out_items = std::move(plan.items);
    }
  }
  *count = (int64_t)out_items.size();
  if (items != nullptr) {
    const int64_t m = std::min<int64_t>(cap, *count);
    for (int64_t i = 0; i < m; i++) items[i] = out_items[(size_t)i];
  }
  return KVX_OK;
}

int extend_attention(kvx_pool* pool, const kvx_batch* batch, const void* q, int32_t num_q_heads, float sm_scale,
                     void* out, float* lse, kvx_stream_t stream) {
  return kvx::attention_call(pool, batch, q, num_q_heads, sm_scale, out, lse, stream, nullptr);
}

}  // extern "C"

int kvx::attention_call(kvx_pool* pool, const kvx_batch* batch, const void* q, int32_t num_q_heads, float sm_scale,
                        void* out, float* lse, kvx_stream_t stream, const FixedScratch* fixed) {
  g_last_error.clear();
  if (int rc = check_pool(pool)) return rc;
  if (int rc = check_heads(num_q_heads, pool->num_kv_heads, pool->head_dim)) return rc;
  if (!(std::isfinite(sm_scale) && sm_scale > 0.f)) return fail(KVX_EINVAL, "sm_scale must be finite and > 0");
  std::vector<int64_t> qo;
  if (int rc = check_batch(batch, qo)) return rc;
  if (qo.back() == 0) return KVX_OK;
  if (!q || !out) return fail(KVX_EINVAL, "q and out must be non-NULL");
  if (int rc = check_align(q, "q")) return rc;
  if (int rc = check_align(out, "out")) return rc;
  if (lse != nullptr && ((uintptr_t)lse & 3u) != 0) return fail(KVX_EINVAL, "lse is not 4-byte aligned");
  hipStream_t s = (hipStream_t)stream;
  CallBuffers buf{pool, fixed};

  if (is_decode_batch(batch, num_q_heads, pool->num_kv_heads))
    return decode_attention(pool, batch, qo, q, num_q_heads, sm_scale, out, lse, s, buf);

  const int D = pool->head_dim;
  const size_t part_bytes = (size_t)kvx::kTileRows * (D + 1) * sizeof(float);
  const size_t dec_part_bytes = (size_t)kvx::kDecodeMaxGroup * (D + 1) * sizeof(float);
  Plan plan;
  kvx::AttnParams p;
  kvx::MergeParams m;
  kvx::CompactPlan compact;
  bool in_args = false;
  std::vector<uint8_t> blob;  // one upload: units, then merges, then the decode units' merges
  bool mixed = is_mixed_batch(batch, num_q_heads, pool->num_kv_heads), packed = false;
  for (;;) {
    PartLimits lim = pool_limits(mixed);
    if (fixed) {
      lim = PartLimits{buf.max_parts(part_bytes), buf.max_parts(dec_part_bytes)};
      // in the fixed scratch, a mixed plan's decode parts have a quarter of the region
      if (mixed) lim = PartLimits{lim.prefill - (lim.prefill + 3) / 4, lim.decode / 4};
    }
    plan = Plan();
    if (int rc = make_plan(batch, qo, num_q_heads, pool->num_kv_heads, D, pool->split_keys, lim, mixed, plan, packed))
      return rc;
    in_args = inline_merges(plan.merges, pool->num_kv_heads, m.plan) && compact_plan(plan, compact);
    if (in_args) break;
    m.plan.n = 0;
    blob = plan_blob(plan.units, plan.merges, plan.dec_merges);
    // what does not fit its region may fit with tiles for the one-token suffixes (fewer units),
    // or else packed (a batch of one long request and 40000 short ones may have most of the
    // short ones on one XCD, and seven paddings to each)
    if (packed || !fixed || blob.size() <= fixed->plan_bytes) break;
    packed = !mixed;
    mixed = false;
    blob.clear();
  }
  if (int rc = buf.check_plan(blob.size())) return rc;
  if (int rc = use_device(pool)) return rc;
  if (validate_mode())
    if (int rc = check_page_ids(pool, batch, s)) return rc;
  if (int rc = buf.bind()) return rc;
  float* parts = nullptr;
  if (plan.n_parts + plan.dec_parts > 0)
    if (int rc = buf.parts((size_t)plan.n_parts * part_bytes + (size_t)plan.dec_parts * dec_part_bytes, s, &parts))
      return rc;
  void* dev = nullptr;
  if (!in_args)
    if (int rc = buf.upload(blob, s, &dev)) return rc;
  p.compact = in_args ? &compact : nullptr;

  p.q = (const uint16_t*)q;
  p.out = (uint16_t*)out;
  p.lse = lse;
  p.k_pool = pool->k;
  p.v_pool = pool->v;
  p.page_ids = batch->page_ids;
  p.units = (const AttnUnit*)dev;
  p.o_part = plan.n_parts ? parts : nullptr;
  p.lse_part = plan.n_parts ? parts + (size_t)plan.n_parts * kvx::kTileRows * D : nullptr;
  p.k_scale = pool->scales_d;
  p.v_scale = pool->scales_d ? pool->scales_d + pool->num_kv_heads : nullptr;
  p.num_q_heads = num_q_heads;
  p.num_kv_heads = pool->num_kv_heads;
  p.group = num_q_heads / pool->num_kv_heads;
  p.tile_tok = kvx::kTileRows / p.group;
  p.scale_log2 = sm_scale * 1.4426950408889634f;
  p.mixed = plan.mixed ? 1 : 0;
  p.d_part = plan.dec_parts ? parts + (size_t)plan.n_parts * (part_bytes / sizeof(float)) : nullptr;
  p.d_lse = plan.dec_parts ? p.d_part + (size_t)plan.dec_parts * kvx::kDecodeMaxGroup * D : nullptr;
  hipError_t e = kvx::launch_extend_attention(p, (int64_t)plan.units.size(), D, pool->kv_dtype == KVX_KV_FP8_E4M3,
                                              pool->scaled_q != 0, s);
  if (e != hipSuccess) return hip_fail(e, "extend_attention kernel launch");
  if (!plan.merges.empty()) {
    m.merges = (const MergeUnit*)((const uint8_t*)dev + plan.units.size() * sizeof(AttnUnit));
    m.o_part = p.o_part;
    m.lse_part = p.lse_part;
    m.out = (uint16_t*)out;
    m.lse = lse;
    m.num_q_heads = num_q_heads;
    m.group = p.group;
    e = kvx::launch_merge(m, (int64_t)plan.merges.size(), D, s);
    if (e != hipSuccess) return hip_fail(e, "merge kernel launch");
  }
  if (!plan.dec_merges.empty()) {
    kvx::DecodeMergeParams dm;
    dm.plan.n = 0;
    dm.merges = (const DecodeMerge*)((const uint8_t*)dev + plan.units.size() * sizeof(AttnUnit) +
                                     plan.merges.size() * sizeof(MergeUnit));
    dm.o_part = p.d_part;
    dm.lse_part = p.d_lse;
    dm.out = (uint16_t*)out;
    dm.lse = lse;
    dm.num_q_heads = num_q_heads;
    dm.group = p.group;
    e = kvx::launch_decode_merge(dm, (int64_t)plan.dec_merges.size(), D, s);
    if (e != hipSuccess) return hip_fail(e, "decode merge kernel launch");
  }
  return buf.done(s, !in_args);
}
