// Host-only checks of how attention calls plan (csrc/kvx_host.cpp), built by
// tests/test_plan_schedule.py.  The argument names the check.  extend_attention_noalloc plans
// before any device work; its scratch has no address here, so that a call whose plan was
// accepted ends with KVX_EHIP and no launch.

#include "kvx_host.cpp"

#include <chrono>
#include <tuple>

namespace kvx {
#define KVX_STUB(name, ...) \
  hipError_t name(__VA_ARGS__) { std::exit(4); }
KVX_STUB(launch_decode, const DecodeParams&, int64_t, int, bool, hipStream_t)
KVX_STUB(launch_decode_merge, const DecodeMergeParams&, int64_t, int, hipStream_t)
KVX_STUB(launch_extend_attention, const AttnParams&, int64_t, int, bool, bool, hipStream_t)
KVX_STUB(launch_merge, const MergeParams&, int64_t, int, hipStream_t)
KVX_STUB(launch_store_kv, const StoreParams&, int64_t, int, bool, hipStream_t)
KVX_STUB(launch_store_kv_rope, const RopeParams&, int64_t, int, bool, bool, hipStream_t)
KVX_STUB(launch_page_move, const PageMoveParams&, int64_t, hipStream_t)
KVX_STUB(launch_page_io, const PageIoParams&, int64_t, int, int, hipStream_t)
}  // namespace kvx

#define CHECK(cond)                                                           \
  do {                                                                        \
    if (!(cond)) {                                                            \
      std::fprintf(stderr, "check failed at line %d: %s\n", __LINE__, #cond); \
      std::exit(3);                                                           \
    }                                                                         \
  } while (0)

namespace {

int no_address(int, void**) { return kvx::report(KVX_EHIP, "no device"); }
const kvx::FixedScratch kFixed{KVX_NOALLOC_PLAN_BYTES, KVX_NOALLOC_PARTS_BYTES, no_address};

struct TestBatch {
  std::vector<int32_t> P, E, indptr{0};
  int32_t ids = 0;
  kvx_batch b{};
  TestBatch(std::vector<int32_t> p, std::vector<int32_t> e) : P(std::move(p)), E(std::move(e)) {
    for (size_t r = 0; r < P.size(); r++)
      indptr.push_back((int32_t)(indptr.back() + ((int64_t)P[r] + E[r] + 15) / 16));
    b.num_reqs = (int32_t)P.size();
    b.prefix_lens = P.data();
    b.extend_lens = E.data();
    b.page_indptr = indptr.data();
    b.page_ids = &ids;
  }
};

int plan_noalloc(const TestBatch& t, int32_t hq, int32_t hkv, int32_t d, const kvx::FixedScratch& fixed = kFixed) {
  kvx_pool pool;
  pool.num_kv_heads = hkv;
  pool.head_dim = d;
  alignas(16) static uint8_t buf[16];
  return kvx::attention_call(&pool, &t.b, buf, hq, 0.125f, buf, nullptr, nullptr, &fixed);
}

template <class F>
double least_us(F&& f, int times) {
  double best = 1e30;
  for (int i = 0; i < times; i++) {
    const auto t0 = std::chrono::steady_clock::now();
    f();
    best = std::min(best, std::chrono::duration<double, std::micro>(std::chrono::steady_clock::now() - t0).count());
  }
  return best;
}

// The allocation-free entry point plans a batch without decode units once.
void check_planned_once() {
  std::vector<int32_t> P, E;
  for (int r = 0; r < 24; r++) {
    P.push_back(10022 + 155 * r);
    E.push_back(124 + 5 * r);
  }
  const TestBatch t(P, E);
  int64_t n = 0;
  double one = 1e30, call = 1e30;
  for (int i = 0; i < 20; i++) {  // in turn, against other work on the machine
    one = std::min(one, least_us([&] { CHECK(extend_attention_plan(&t.b, 8, 1, 128, 0, nullptr, 0, &n) == KVX_OK); }, 5));
    call = std::min(call, least_us([&] { CHECK(plan_noalloc(t, 8, 1, 128) == KVX_EHIP); }, 5));
  }
  std::printf("plan %.0f us, call %.0f us\n", one, call);
  CHECK(call < 1.7 * one);  // planned twice: 2.5
}

// The search for a split costs at most as much as three plans of the split it found (many
// tiles of one KV head, where a trial schedule has the most units).
void check_search_time() {
  for (const auto& [hq, n, p, step, e] : std::vector<std::tuple<int32_t, int, int32_t, int32_t, int32_t>>{
           {8, 24, 10022, 155, 124}, {32, 8, 2366, 5000, 230}, {8, 7, 2593, 2350, 1050}}) {
    std::vector<int32_t> P, E;
    for (int r = 0; r < n; r++) {
      P.push_back(p + step * r);
      E.push_back(e + 5 * r);
    }
    const TestBatch t(P, E);
    int64_t count = 0;
    CHECK(extend_attention_plan(&t.b, hq, 1, 128, 0, nullptr, 0, &count) == KVX_OK);
    std::vector<kvx_work_item> items((size_t)count);
    CHECK(extend_attention_plan(&t.b, hq, 1, 128, 0, items.data(), count, &count) == KVX_OK);
    int32_t split = 0;
    for (const kvx_work_item& i : items)
      if (i.part >= 0 && i.key_begin == 0) split = i.key_end;
    CHECK(split > 0);
    double forced = 1e30, found = 1e30;
    for (int i = 0; i < 20; i++) {
      forced = std::min(forced, least_us([&] { extend_attention_plan(&t.b, hq, 1, 128, split, nullptr, 0, &count); }, 5));
      found = std::min(found, least_us([&] { extend_attention_plan(&t.b, hq, 1, 128, 0, nullptr, 0, &count); }, 5));
    }
    std::printf("forced %.0f us, found %.0f us\n", forced, found);
    CHECK(found < 4.0 * forced);
  }
}

// With few parts allowed, the split chosen makes a schedule within a tenth of the best one
// among all lengths that keep within them.
void check_limited_splits() {
  struct Shape {
    int32_t hq, hkv, d, n, p0, p1, e0, e1;
  };
  const Shape shapes[] = {{32, 8, 128, 3, 37701, 48480, 313, 494}, {16, 1, 128, 5, 29560, 44412, 424, 1018},
                          {8, 1, 128, 19, 34942, 48111, 233, 250}, {40, 10, 128, 3, 46465, 49414, 298, 339},
                          {4, 2, 64, 2, 21610, 88566, 90, 3157},   {64, 8, 128, 40, 1000, 60000, 10, 300}};
  int limited = 0;
  for (const Shape& h : shapes) {
    const int32_t tile_tok = kvx::kTileRows / (h.hq / h.hkv);
    std::vector<Tile> tiles;
    for (int32_t r = 0; r < h.n; r++) {
      const int64_t P = h.p0 + (int64_t)(h.p1 - h.p0) * r / (h.n - 1), E = h.e0 + (int64_t)(h.e1 - h.e0) * (r * 7 % h.n) / (h.n - 1);
      for (int64_t t0 = (E - 1) / tile_tok * tile_tok; t0 >= 0; t0 -= tile_tok) {
        const int64_t n = std::min<int64_t>(tile_tok, E - t0);
        tiles.push_back(Tile{r, (int32_t)t0, (int32_t)n, P + t0 + n, P + t0});
      }
    }
    const int64_t max_parts = KVX_NOALLOC_PARTS_BYTES / ((int64_t)kvx::kTileRows * (h.d + 1) * 4);
    Trials trial(tiles, h.hkv, tile_tok, h.d == 128 ? kUnitCosts128 : kUnitCosts64, Filler{});
    const int64_t split = choose_split(tiles, h.hkv, tile_tok, h.d, Filler{}, max_parts);
    CHECK(trial.cut(split) * h.hkv <= max_parts);
    const double got = trial.length(1e300);
    trial.cut(0);
    double best = trial.length(1e300);
    int64_t most = 0;
    for (int64_t len = 4; len * 64 <= h.p1 + h.e1; len++) {
      const int64_t parts = trial.cut(len * 64) * h.hkv;
      most = std::max(most, parts);
      if (parts <= max_parts) best = std::min(best, trial.length(1e300));
    }
    limited += choose_split(tiles, h.hkv, tile_tok, h.d, Filler{}, kMaxParts) != split;
    std::printf("%d/%d heads: schedule %.0f, best %.0f, split %lld\n", h.hq, h.hkv, got, best, (long long)split);
    CHECK(got <= 1.1 * best);
  }
  CHECK(limited >= 3);
}

// The allocation-free entry point takes every batch whose units alone fit its plan region.
void check_all_that_fits() {
  struct Shape {
    int32_t hq, hkv, P, E, n, p, e;  // one long request, n short ones
  };
  const int64_t room = KVX_NOALLOC_PLAN_BYTES / (int64_t)sizeof(AttnUnit);
  int packed = 0;
  for (const Shape& h : {Shape{8, 1, 98740, 242150, 116000, 60, 2}, Shape{8, 1, 131072, 75000, 60000, 40, 3},
                         Shape{32, 1, 2104, 182903, 103000, 1000, 2}, Shape{8, 2, 98979, 15359, 78000, 60, 9},
                         Shape{4, 2, 100000, 180000, 80000, 30, 3}, Shape{8, 8, 4295, 2000, 32000, 30, 2}}) {
    std::vector<int32_t> P{h.P}, E{h.E};
    const int32_t tile_tok = kvx::kTileRows / (h.hq / h.hkv);
    int64_t units = ((int64_t)h.E + tile_tok - 1) / tile_tok * h.hkv;
    for (int32_t r = 0; r < h.n; r++) {
      P.push_back(r % h.p);
      E.push_back(1 + r % h.e);
      units += h.hkv;
    }
    const TestBatch t(P, E);
    int64_t n = 0;
    CHECK(units <= room && extend_attention_plan(&t.b, h.hq, h.hkv, 128, 0, nullptr, 0, &n) == KVX_OK);
    packed += n > room;
    std::printf("%lld units, %lld with padding\n", (long long)units, (long long)n);
    CHECK(plan_noalloc(t, h.hq, h.hkv, 128) == KVX_EHIP);
  }
  CHECK(packed >= 2);
  // mixed: the merges of one chunked decode are too much, tiles for all fit to the last unit
  std::vector<int32_t> P(32768, 100), E(32768, 1);
  P[0] = 100000;
  E[1] = 2;
  const TestBatch t(P, E);
  CHECK(is_mixed_batch(&t.b, 8, 8));
  CHECK(plan_noalloc(t, 8, 8, 128) == KVX_EHIP);
  const kvx::FixedScratch less{KVX_NOALLOC_PLAN_BYTES - 32, KVX_NOALLOC_PARTS_BYTES, no_address};
  CHECK(plan_noalloc(t, 8, 8, 128, less) == KVX_EUNSUPPORTED);
}

// The partial results of a mixed batch, of both kinds together, stay within those of kMaxParts
// tiles (the 2 GiB that kvx.h states).
void check_bound_on_parts() {
  const TestBatch t({64 * 16000, 64 * 16000, 64 * 300}, {32, 1, 1});
  int64_t n = 0;
  CHECK(extend_attention_plan(&t.b, 8, 1, 128, 64, nullptr, 0, &n) == KVX_OK);
  std::vector<kvx_work_item> items((size_t)n);
  CHECK(extend_attention_plan(&t.b, 8, 1, 128, 64, items.data(), n, &n) == KVX_OK);
  int64_t prefill = 0, decode = 0;
  for (const kvx_work_item& i : items)
    if (i.part >= 0) (i.req == 0 ? prefill : decode) += 1;
  std::printf("%lld prefill parts, %lld decode parts\n", (long long)prefill, (long long)decode);
  CHECK(prefill > 0 && decode > 0);
  CHECK(prefill * kvx::kTileRows + decode * kvx::kDecodeMaxGroup <= kMaxParts * kvx::kTileRows);
}

}  // namespace

int main(int argc, char** argv) {
  const std::string what = argv[argc - 1];
  if (what == "once") check_planned_once();
  else if (what == "search") check_search_time();
  else if (what == "limits") check_limited_splits();
  else if (what == "fits") check_all_that_fits();
  else if (what == "bound") check_bound_on_parts();
  else return 2;
  std::printf("passed\n");
  return 0;
}
