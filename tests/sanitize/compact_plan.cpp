// Host-only check of the plans that travel in kernel arguments (csrc/kvx_host.cpp), built
// with AddressSanitizer and UndefinedBehaviorSanitizer by tests/test_plan_schedule.py: what
// the arguments are expanded to must be, entry by entry, what would have been uploaded.
// The prefill expansion is the kernels' own (unit_from_plan); the decode units' and the
// merges' is worked out here from their definition.

#include "kvx_host.cpp"

#include <random>

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

int main(int argc, char** argv) {
  std::mt19937_64 rng(77);
  auto uni = [&](int64_t lo, int64_t hi) { return std::uniform_int_distribution<int64_t>(lo, hi)(rng); };
  int64_t compact_plans = 0, grouped = 0, split = 0, decode_plans = 0, merged = 0, uploaded = 0;
  for (int it = 0; it < std::atoi(argv[argc - 1]); it++) {
    const bool decode = it % 3 == 0;
    const int R = (int)uni(1, 24), hkv = (int)std::vector<int>{1, 2, 3, 8, 16}[(size_t)uni(0, 4)];
    const int g = (int)std::vector<int>{1, 2, 4, 8, 16}[(size_t)uni(0, 4)];
    const int64_t pmax = std::vector<int64_t>{50, 2000, 60000}[(size_t)uni(0, 2)];
    const int64_t emax = std::vector<int64_t>{1, 40, 700, 3000}[(size_t)uni(0, 3)];
    std::vector<int32_t> P, E, indptr{0};
    for (int r = 0; r < R; r++) {
      P.push_back((int32_t)uni(0, pmax));
      E.push_back((int32_t)(decode ? uni(0, 1) : uni(0, emax)));
      indptr.push_back(indptr.back() + (P.back() + E.back() + 15) / 16);
    }
    int32_t dummy = 0;
    kvx_batch b{};
    b.num_reqs = R;
    b.prefix_lens = P.data();
    b.extend_lens = E.data();
    b.page_indptr = indptr.data();
    b.page_ids = &dummy;
    std::vector<int64_t> qo;
    CHECK(check_batch(&b, qo) == KVX_OK);
    const int32_t forced = uni(0, 2) ? 0 : (int32_t)(64 * uni(1, 40));
    if (decode) {
      DecodePlan plan;
      CHECK(make_decode_plan(&b, qo, hkv, forced, kMaxParts, plan) == KVX_OK);
      static kvx::InlinePlan<DecodeUnit> in;
      kvx::InlineMerges<DecodeMerge> im;
      if (inline_units(plan.units, in) && in.n > 0) {
        decode_plans++;
        CHECK((size_t)in.n * in.heads == plan.units.size());
        for (size_t i = 0; i < plan.units.size(); i++) {
          DecodeUnit u = in.unit[i / in.heads];
          const int32_t h = (int32_t)(i % in.heads);
          u.head += h;
          if (u.part >= 0) u.part += h * u.req;
          u.req = plan.units[i].req;
          CHECK(std::memcmp(&u, &plan.units[i], sizeof u) == 0);
        }
      }
      if (inline_merges(plan.merges, hkv, im)) CHECK((size_t)im.n * im.heads == plan.merges.size());
      continue;
    }
    Plan plan;
    CHECK(make_plan(&b, qo, hkv * g, hkv, 128, forced, PartLimits{kMaxParts, kMaxParts},
                    uni(0, 1) == 1 && is_mixed_batch(&b, hkv * g, hkv), plan) == KVX_OK);
    static kvx::CompactPlan c;
    if (compact_plan(plan, c)) {
      compact_plans++;
      grouped += c.heads > 1;
      split += !plan.merges.empty();
      CHECK(!plan.mixed && (size_t)c.n == plan.units.size());
      CHECK(6 * (size_t)c.n_tiles + ((size_t)c.n + c.heads - 1) / c.heads <= (size_t)kvx::kPlanWords);
      for (int i = 0; i < c.n; i++) {
        AttnUnit u = kvx::unit_from_plan(c, (const uint32_t*)c.words, i), v = plan.units[(size_t)i];
        if (v.key_end <= v.key_begin) {
          CHECK(u.key_end <= u.key_begin);
          continue;
        }
        u.req = v.req;  // no kernel uses it
        CHECK(std::memcmp(&u, &v, sizeof u) == 0);
      }
    } else {
      uploaded++;
    }
    kvx::InlineMerges<MergeUnit> im;
    if (inline_merges(plan.merges, hkv, im)) {
      CHECK((size_t)im.n * im.heads == plan.merges.size());
      merged += im.n > 0;
    }
  }
  CHECK(compact_plans > 0 && grouped > 0 && split > 0 && decode_plans > 0 && merged > 0 && uploaded > 0);
  std::printf("passed: %lld compact (%lld by eights, %lld split), %lld decode, %lld merge lists, %lld uploaded\n",
              (long long)compact_plans, (long long)grouped, (long long)split, (long long)decode_plans,
              (long long)merged, (long long)uploaded);
  return 0;
}
