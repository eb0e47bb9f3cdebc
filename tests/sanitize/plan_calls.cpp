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
  CHECK(call < 1.5 * one);
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

}  // namespace

int main(int argc, char** argv) {
  const std::string what = argv[argc - 1];
  if (what == "once") check_planned_once();
  else if (what == "search") check_search_time();
  else return 2;
  std::printf("passed\n");
  return 0;
}
