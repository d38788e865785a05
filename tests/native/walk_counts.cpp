// count_walks and count_dkv_walks (csrc/plan.hpp), which sum by segment, against the items that plan_fwd and plan_dkv list: random chunks and all block sizes in use.
#include <algorithm>
#include <cstdio>
#include <random>

#include "../../paper_2509_21275_amd/csrc/plan.hpp"

#define REQUIRE(x) do { if (!(x)) { std::printf("line %d: %s\n", __LINE__, #x); return 1; } } while (0)
using namespace chunk_attn;

static int one(const std::vector<chunk_attn_seg>& segs, int heads, int kv_heads) {
  const chunk_attn_desc d{heads, kv_heads, 128, segs.back().q_start + segs.back().q_len, segs.back().kv_start + segs.back().kv_len, (int)segs.size(), segs.data(), 0.1f};
  REQUIRE(validate(&d) == CHUNK_ATTN_OK);
  for (int rows : {32, 64, 128, 256}) {
    int64_t items = 0, stages = 0, longest = 0;
    for (const FwdItem& it : plan_fwd(&d, rows)) {
      const int64_t n = walk_stages(it.n0, it.q_rows);
      ++items;
      stages += n;
      longest = std::max(longest, n);
    }
    const Walks w = count_walks(&d, rows);
    REQUIRE(w.items == items && w.stages == stages && w.longest == longest);
    int64_t largest = 0;
    for (const auto& s : segs) largest = std::max<int64_t>(largest, (s.q_len + rows - 1) / rows);
    REQUIRE(w.largest == largest);
  }
  for (int keys : {32, 64, 128, 256}) {
    int64_t items = 0, steps = 0, longest = 0;
    for (const DkvItem& it : plan_dkv(&d, keys)) {
      const int64_t n = (int64_t)(it.n_qt - it.qt_first) * (heads / kv_heads);
      ++items;
      steps += n;
      longest = std::max(longest, n);
    }
    const Walks w = count_dkv_walks(&d, keys);
    REQUIRE(w.items == items && w.stages == steps && w.longest == longest);
    int64_t largest = 0;
    for (const auto& s : segs) largest = std::max<int64_t>(largest, (s.kv_len + keys - 1) / keys);
    REQUIRE(w.largest == largest);
  }
  return 0;
}

int main() {
  std::mt19937 rng(11);
  auto up_to = [&](int n) { return (int)(rng() % n); };
  for (int rep = 0; rep < 4000; ++rep) {
    std::vector<chunk_attn_seg> segs;
    int q = 0, kv = 0;
    for (int n = 1 + up_to(6); n > 0; --n) {
      const int edge = 32 << up_to(5), q_len = std::max(1, up_to(2) ? 1 + up_to(1200) : edge + up_to(3) - 1), ctx = up_to(3) == 0 ? 0 : up_to(2) ? up_to(3000) : edge + up_to(3) - 1;
      kv += up_to(3);
      segs.push_back(chunk_attn_seg{q, q_len, kv, q_len + ctx});
      q += q_len;
      kv += q_len + ctx;
    }
    const int kv_heads = 1 + up_to(4);
    if (one(segs, kv_heads * (1 + up_to(8)), kv_heads)) return 1;
  }
  std::printf("ok\n");
  return 0;
}
