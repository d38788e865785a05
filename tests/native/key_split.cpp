// Cutting the walks of query-stationary work items over the keys (csrc/plan.hpp): random chunks, every target.
//   * the pieces of an item are consecutive, begin on even stages, cover its keys once and in order;
//   * the first key of a piece is visible to the item's first row, every piece but the last is visible whole to every row;
//   * slots of partial results are handed out in order, to pieces of cut items only;
//   * choose_key_split and refine_bwd_split count what cut_items makes and respect their limits; choose_key_split cuts chunks with few long
//     walks and no others.
#include <algorithm>
#include <chrono>
#include <cstdio>
#include <random>

#include "../../paper_2509_21275_amd/csrc/plan.hpp"

#define REQUIRE(x) do { if (!(x)) { std::printf("line %d: %s\n", __LINE__, #x); return 1; } } while (0)
using namespace chunk_attn;

template <class Item>
static int check(const std::vector<Item>& wholes, const std::vector<Item>& items, int target, int64_t* parts_out) {
  size_t x = 0;
  int32_t part = 0;
  for (size_t w = 0; w < wholes.size(); ++w) {
    const Item& whole = wholes[w];
    const int last_key = whole.kv_row0 + whole.n0 + whole.q_rows - 1;  // behind the keys the last row sees
    const int n = piece_count(walk_stages(whole.n0, whole.q_rows), whole.n0, target);
    int next = whole.kv_row0;
    for (int k = 0; k < n; ++k, ++x) {
      REQUIRE(x < items.size());
      const Item& it = items[x];
      REQUIRE(it.q_row0 == whole.q_row0 && it.q_rows == whole.q_rows);
      REQUIRE(it.kv_row0 == next && (it.kv_row0 - whole.kv_row0) % (2 * kStageKeys) == 0);
      REQUIRE(it.n0 == whole.n0 - (it.kv_row0 - whole.kv_row0) && it.n0 >= 1);
      const int end = it.kv_row0 + std::min(it.n0 + it.q_rows - 1, it.keys);
      if (k + 1 < n) {
        REQUIRE(it.keys <= it.n0 && it.keys % kStageKeys == 0 && end == it.kv_row0 + it.keys);
      } else {
        REQUIRE(end == last_key);
      }
      next = end;
      REQUIRE(it.part == (n > 1 ? part : -1));
      if (n > 1) ++part;
    }
  }
  REQUIRE(x == items.size());
  *parts_out = part;
  return 0;
}

static int one(const std::vector<chunk_attn_seg>& segs, int heads, int kv_heads, int expect_cut) {
  int tq = 0, tkv = 0;
  for (const auto& s : segs) { tq = s.q_start + s.q_len; tkv = s.kv_start + s.kv_len; }
  chunk_attn_desc d{heads, kv_heads, 128, tq, tkv, (int)segs.size(), segs.data(), 0.1f};
  REQUIRE(validate(&d) == CHUNK_ATTN_OK);
  const int group = heads / kv_heads;
  int h = 1;
  while (h * 2 <= 4 && group % (h * 2) == 0) h *= 2;
  const int rows = 256 / h, inner = kv_heads * (group / h);
  for (int target : {0, 1, 8, 9, 13, 40, 100000}) {
    int64_t parts = 0;
    auto w = plan_fwd(&d, rows);
    const auto items = cut_items(w, target);
    if (check(w, items, target, &parts)) return 1;
    size_t x = 0;
    for (size_t i = 0; i < w.size(); ++i) {
      REQUIRE(w[i].pieces >= 1 && (w[i].part >= 0) == (w[i].pieces > 1) && (w[i].part < 0 || w[i].part == items[x].part));
      for (int k = 0; k < w[i].pieces; ++k, ++x) REQUIRE(items[x].q_row0 == w[i].q_row0);
    }
    const auto q = plan_dq(&d, rows);
    std::vector<DqItem> cut;
    if (check(q, cut_items(q, target, &cut), target, &parts)) return 1;
    int64_t sum = 0;
    for (const auto& c : cut) { REQUIRE(c.pieces > 1 && c.part == sum); sum += c.pieces; }
    REQUIRE(sum == parts);
  }
  for (int target : {0, 1, 2, 5, 100000}) {  // key-stationary: every piece a run of its walk's query tiles
    const auto w = plan_dkv(&d, 128);
    std::vector<DkvItem> cut;
    const auto items = cut_items(w, target, &cut);
    size_t n_items = 0;
    int32_t part = 0;
    for (const auto& whole : w) {
      std::vector<DkvItem> mine;
      for (const auto& it : items) if (it.kv_row0 == whole.kv_row0) mine.push_back(it);
      std::sort(mine.begin(), mine.end(), [](const DkvItem& a, const DkvItem& b) { return a.qt_first < b.qt_first; });
      int next = whole.qt_first;
      for (const auto& it : mine) {
        REQUIRE(it.qt_first == next && it.n_qt > it.qt_first && it.q_len == whole.q_len && it.q_tile0 == whole.q_tile0);
        REQUIRE(it.part == (mine.size() > 1 ? part : -1) && !it.reverse);
        if (mine.size() > 1) ++part;
        next = it.n_qt;
      }
      REQUIRE(next == whole.n_qt);
      n_items += mine.size();
    }
    REQUIRE(n_items == items.size());
    int32_t sum = 0;
    for (const auto& c : cut) { REQUIRE(c.pieces > 1 && c.part == sum); sum += c.pieces; }
    REQUIRE(sum == part);
    for (size_t i = 1; i < items.size(); ++i) REQUIRE(items[i].n_qt - items[i].qt_first <= items[i - 1].n_qt - items[i - 1].qt_first);
  }
  for (int64_t limit : {(int64_t)0, (int64_t)5, (int64_t)1 << 40}) {
    const KeySplit k = choose_tile_split(&d, 128, 256, limit);
    REQUIRE(k.parts <= limit);
    if (k.target > 0) {
      std::vector<DkvItem> cut;
      const auto items = cut_items(plan_dkv(&d, 128), k.target, &cut);
      int64_t parts = 0;
      for (const auto& c : cut) parts += c.pieces;
      REQUIRE(k.pieces == (int64_t)items.size() && k.parts == parts && parts > 0);
    }
  }
  for (int64_t limit : {(int64_t)3, (int64_t)40, (int64_t)1 << 40}) {  // both kinds of a backward: kinds that are whole by themselves stay whole
    const KeySplit q0 = choose_key_split(&d, rows, inner, 256, limit / inner), k0 = choose_tile_split(&d, 128, 256, limit / kv_heads);
    KeySplit q1 = q0, k1 = k0;
    refine_bwd_split(&d, rows, inner, 128, 256, 2 * limit, &q1, &k1);
    REQUIRE((q1.target == 0 || q0.target > 0) && (k1.target == 0 || k0.target > 0));
    REQUIRE(q1.parts * inner <= 2 * limit && k1.parts * kv_heads <= 2 * limit);
    std::vector<DqItem> qcut;
    std::vector<DkvItem> kcut;
    const auto qi = cut_items(plan_dq(&d, rows), q1.target, &qcut);
    const auto ki = cut_items(plan_dkv(&d, 128), k1.target, &kcut);
    int64_t qp = 0, kp = 0;
    for (const auto& c : qcut) qp += c.pieces;
    for (const auto& c : kcut) kp += c.pieces;
    REQUIRE(qp == q1.parts && kp == k1.parts && (q1.target == 0 || q1.pieces == (int64_t)qi.size()) && (k1.target == 0 || k1.pieces == (int64_t)ki.size()));
  }
  for (int64_t limit : {(int64_t)0, (int64_t)3, (int64_t)1 << 40}) {
    const KeySplit k = choose_key_split(&d, rows, inner, 256, limit);
    REQUIRE(k.parts <= limit);
    if (limit == 0) REQUIRE(k.target == 0);
    if (limit > 3 && expect_cut >= 0) REQUIRE((k.target > 0) == (expect_cut > 0));
    if (k.target > 0) {
      int64_t parts = 0;
      auto w = plan_fwd(&d, rows);
      const auto items = cut_items(w, k.target);
      if (check(w, items, k.target, &parts)) return 1;
      REQUIRE(k.parts == parts && k.pieces == (int64_t)items.size() && k.parts > 0);
    }
  }
  return 0;
}

// What a backward's launch runs is what the estimate for both kinds together finds best: whole walks though one kind by itself would be cut, the cuts
// of each kind by itself, or others (targets in stages and tiles; 0: whole).
static int joint(int q, int ctx, int heads, int kv_heads, int dq_alone, int dkv_alone, int dq, int dkv) {
  chunk_attn_seg s{0, q, 0, ctx + q};
  chunk_attn_desc d{heads, kv_heads, 128, q, ctx + q, 1, &s, 0.1f};
  const int group = heads / kv_heads;
  int h = 1;
  while (h * 2 <= 8 && group % (h * 2) == 0) h *= 2;
  const int rows = 256 / h, inner = kv_heads * (group / h);
  const int64_t room = (int64_t)fused_num_bufs(&d, 128) * heads * ((q + 31) / 32) / 8;  // partial results as large as the float32 dQ tiles
  KeySplit a = choose_key_split(&d, rows, inner, 256, room / inner), b = choose_tile_split(&d, 128, 256, room / kv_heads);
  REQUIRE(a.target == dq_alone && b.target == dkv_alone);
  refine_bwd_split(&d, rows, inner, 128, 256, std::max<int64_t>(room, 512), &a, &b);
  if (a.target != dq || b.target != dkv) std::printf("%d queries behind %d keys: %d and %d\n", q, ctx, a.target, b.target);
  REQUIRE(a.target == dq && b.target == dkv && (a.parts > 0) == (dq > 0) && (b.parts > 0) == (dkv > 0));
  return 0;
}

// Chunks with more blocks than are ever cut cost a call no list of their walks (of a million blocks here, tens of milliseconds).
static int many_blocks_take_no_time() {
  chunk_attn_seg s{0, 1 << 27, 0, 1 << 27};
  chunk_attn_desc d{8, 8, 128, 1 << 27, 1 << 27, 1, &s, 0.1f};
  double ms = 1e9;
  for (int i = 0; i < 5; ++i) {
    const auto t0 = std::chrono::steady_clock::now();
    KeySplit q = choose_key_split(&d, 256, 8, 256, 1000), k = choose_tile_split(&d, 128, 256, 1000);
    refine_bwd_split(&d, 256, 8, 128, 256, 1000, &q, &k);
    REQUIRE(q.target == 0 && k.target == 0);
    ms = std::min(ms, std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count());
  }
  REQUIRE(ms < 1.0);
  return 0;
}

int main() {
  std::mt19937 rng(7);
  auto uni = [&](int a, int b) { return std::uniform_int_distribution<int>(a, b)(rng); };
  for (int n = 0; n < 400; ++n) {
    std::vector<chunk_attn_seg> segs;
    int tq = 0, tkv = 0;
    for (int i = uni(1, 6); i > 0; --i) {
      const int q = uni(0, 1) ? uni(1, 70) : uni(1, 1500), c = uni(0, 2) ? 0 : uni(1, 6000);
      segs.push_back({tq, q, tkv, c + q});
      tq += q;
      tkv += c + q + uni(0, 3);
    }
    const int kv = 1 << uni(0, 3), g = uni(1, 8);
    if (one(segs, kv * g, kv, -1)) { std::printf("case %d\n", n); return 1; }
  }
  if (one({{0, 1024, 0, 32768}}, 32, 8, 1)) return 1;    // half as many items as compute units, long walks
  if (one({{0, 1, 0, 1100}}, 8, 2, 1)) return 1;
  if (one({{0, 8192, 0, 32768}}, 32, 8, 0)) return 1;    // four items per compute unit
  if (one({{0, 100, 0, 100}, {100, 60, 100, 60}}, 8, 8, 0)) return 1;  // walks too short to cut
  if (joint(483, 1954, 32, 8, 39, 0, 0, 0) || joint(3823, 5291, 8, 2, 143, 60, 143, 60) || joint(6863, 10, 8, 2, 72, 31, 0, 72)) return 1;
  if (many_blocks_take_no_time()) return 1;
  std::printf("ok\n");
  return 0;
}
