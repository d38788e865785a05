#include "plan.hpp"

#include <algorithm>
#include <cmath>
#include <numeric>

namespace chunk_attn {

int validate(const chunk_attn_desc* d) {
  if (!d || !d->segments) return CHUNK_ATTN_INVALID_ARG;
  if (d->num_q_heads <= 0 || d->num_kv_heads <= 0 || d->head_dim <= 0 || d->total_q <= 0 || d->total_kv <= 0 ||
      d->num_segments <= 0)
    return CHUNK_ATTN_INVALID_ARG;
  if (!(d->softmax_scale > 0.0f) || !std::isfinite(d->softmax_scale)) return CHUNK_ATTN_INVALID_ARG;
  if (d->head_dim != 64 && d->head_dim != 96 && d->head_dim != 128 && d->head_dim != 256) return CHUNK_ATTN_UNSUPPORTED;
  if (d->num_q_heads % d->num_kv_heads != 0) return CHUNK_ATTN_UNSUPPORTED;
  int64_t q_next = 0, kv_next = 0;
  for (int t = 0; t < d->num_segments; ++t) {
    const chunk_attn_seg& s = d->segments[t];
    if (s.q_len < 1 || s.kv_len < s.q_len) return CHUNK_ATTN_BAD_SEGMENT;
    if (s.q_start != q_next) return CHUNK_ATTN_BAD_SEGMENT;  // in order, back to back, from row 0
    if (s.kv_start < kv_next) return CHUNK_ATTN_BAD_SEGMENT; // in order, no overlap
    q_next = (int64_t)s.q_start + s.q_len;
    kv_next = (int64_t)s.kv_start + s.kv_len;
    if (q_next > d->total_q || kv_next > d->total_kv) return CHUNK_ATTN_BAD_SEGMENT;
  }
  if (q_next != d->total_q) return CHUNK_ATTN_BAD_SEGMENT;
  return CHUNK_ATTN_OK;
}

int64_t pair_count(const chunk_attn_desc* d) {
  int64_t n = 0;
  for (int t = 0; t < d->num_segments; ++t) {
    const int64_t s = d->segments[t].q_len, C = (int64_t)d->segments[t].kv_len - s;
    n += s * C + s * (s + 1) / 2;
  }
  return n;
}

int64_t count_tiles(const chunk_attn_desc* d, bool kv, int width) {
  int64_t n = 0;
  for (int t = 0; t < d->num_segments; ++t)
    n += ((kv ? d->segments[t].kv_len : d->segments[t].q_len) + width - 1) / width;
  return n;
}

std::vector<TileJob> query_tile_jobs(const chunk_attn_desc* d, int width) {
  std::vector<TileJob> jobs;
  for (int t = 0; t < d->num_segments; ++t) {
    const chunk_attn_seg& s = d->segments[t];
    for (int32_t r = 0; r < s.q_len; r += width) {
      TileJob j;
      j.src_row0 = s.q_start + r;
      j.valid_rows = std::min<int32_t>(width, s.q_len - r);
      j.image = (int32_t)jobs.size();
      j.pad = 0;
      jobs.push_back(j);
    }
  }
  return jobs;
}

// Order of the query-stationary work items: sequence by sequence, the sequence with the most keys first, and inside a
// sequence the query tile that walks the most keys first.  The workgroups of an XCD then work on neighbouring tiles of
// one sequence and share its K / V stream in the L2, the long sequences still start first, and every sequence ends in
// short items that fill the tail (the workgroups balance the rest by taking blocks from each other's queues).
// Measured against "longest walk first over the whole chunk": +1.7 % on the packed 64K chunk, nothing on the others.
template <class Item>
static void by_sequence_then_walk(const chunk_attn_desc* d, std::vector<Item>& items) {
  std::vector<int32_t> keys_of(d->total_kv + 1, 0);  // by the first key row of a segment: its number of keys
  for (int t = 0; t < d->num_segments; ++t) keys_of[d->segments[t].kv_start] = d->segments[t].kv_len;
  std::stable_sort(items.begin(), items.end(), [&](const Item& a, const Item& b) {
    const int32_t ka = keys_of[a.kv_row0], kb = keys_of[b.kv_row0];
    if (ka != kb) return ka > kb;
    if (a.kv_row0 != b.kv_row0) return a.kv_row0 < b.kv_row0;
    return (int64_t)a.n0 + a.q_rows > (int64_t)b.n0 + b.q_rows;
  });
}

std::vector<FwdItem> plan_fwd(const chunk_attn_desc* d, int tile_rows) {
  std::vector<FwdItem> items;
  for (int t = 0; t < d->num_segments; ++t) {
    const chunk_attn_seg& s = d->segments[t];
    const int32_t C = s.kv_len - s.q_len;
    for (int32_t i0 = 0; i0 < s.q_len; i0 += tile_rows) {
      FwdItem it{};
      it.q_row0 = s.q_start + i0;
      it.q_rows = std::min<int32_t>(tile_rows, s.q_len - i0);
      it.kv_row0 = s.kv_start;
      it.n0 = C + i0 + 1;
      it.keys = s.kv_len;
      it.part = -1;
      items.push_back(it);
    }
  }
  by_sequence_then_walk(d, items);
  for (FwdItem& it : items) it.pieces = 1;
  return items;
}

std::vector<DqItem> plan_dq(const chunk_attn_desc* d, int tile_rows) {
  std::vector<DqItem> items;
  int32_t q_tile0 = 0;
  for (int t = 0; t < d->num_segments; ++t) {
    const chunk_attn_seg& s = d->segments[t];
    const int32_t C = s.kv_len - s.q_len;
    for (int32_t i0 = 0; i0 < s.q_len; i0 += tile_rows) {
      DqItem it{};
      it.q_row0 = s.q_start + i0;
      it.q_rows = std::min<int32_t>(tile_rows, s.q_len - i0);
      it.kv_row0 = s.kv_start;
      it.n0 = C + i0 + 1;
      it.q_slot0 = q_tile0 * 64 + i0;
      it.keys = s.kv_len;
      it.part = -1;
      items.push_back(it);
    }
    q_tile0 += (s.q_len + 63) / 64;
  }
  by_sequence_then_walk(d, items);
  return items;
}

// (Part of every call, so by segment: the tiles of a segment walk ceil(C / 32) + r, + 2 r ... stages, r 32-row units to a tile, and the last one all of its keys.)
Walks count_walks(const chunk_attn_desc* d, int tile_rows) {
  Walks w;
  const int64_t r = tile_rows / 32;
  for (int t = 0; t < d->num_segments; ++t) {
    const chunk_attn_seg& s = d->segments[t];
    const int64_t n = ((int64_t)s.q_len + tile_rows - 1) / tile_rows, before = ((int64_t)s.kv_len - s.q_len + 31) / 32, last = ((int64_t)s.kv_len + 31) / 32;
    w.largest = std::max(w.largest, n);
    w.items += n;
    w.stages += (n - 1) * before + r * (n * (n - 1) / 2) + last;
    w.longest = std::max(w.longest, last);
  }
  return w;
}

std::vector<ShareBlock> share_blocks(const chunk_attn_desc* d, bool keys) {
  std::vector<ShareBlock> out;
  const int group = d->num_q_heads / d->num_kv_heads;
  for (int t = 0; t < d->num_segments; ++t) {
    const chunk_attn_seg& s = d->segments[t];
    const int32_t C = s.kv_len - s.q_len, n_qt = (s.q_len + 31) / 32;
    for (int32_t x = 0; 32 * x < (keys ? s.kv_len : s.q_len); ++x)
      out.push_back({t, x, keys ? (int64_t)(n_qt - std::max(0, 32 * x - C) / 32) * group : walk_stages(C + 32 * x + 1, std::min(32, s.q_len - 32 * x))});
  }
  std::stable_sort(out.begin(), out.end(), [](const ShareBlock& a, const ShareBlock& b) { return a.steps > b.steps; });
  return out;
}

// (By segment, too: blocks that begin inside the context, or where it ends, walk all query tiles, the others keys / 32 fewer from one to the next.)
Walks count_dkv_walks(const chunk_attn_desc* d, int keys) {
  Walks w;
  const int64_t group = d->num_q_heads / d->num_kv_heads, r = keys / 32;
  for (int t = 0; t < d->num_segments; ++t) {
    const chunk_attn_seg& s = d->segments[t];
    const int64_t C = (int64_t)s.kv_len - s.q_len, n_qt = ((int64_t)s.q_len + 31) / 32, n = ((int64_t)s.kv_len + keys - 1) / keys;
    const int64_t whole = C / keys + 1, part = n - whole;  // (n >= whole: the last block begins behind C / keys blocks)
    w.longest = std::max(w.longest, n_qt * group);
    w.largest = std::max(w.largest, n);
    w.items += n;
    // block j begins at key keys j, behind ceil(C / 32) query tiles' worth of context: it lacks r j - ceil(C / 32) of the query tiles
    w.stages += (n * n_qt - (r * ((whole + n - 1) * part / 2) - part * ((C + 31) / 32))) * group;
  }
  return w;
}

// The estimate behind the cuts, in steps of a workgroup (about a microsecond each).  A block costs its steps plus
// kStart for filling the pipeline and writing its rows; a piece kPart more for its float32 rows (twice the bytes).  The
// blocks of queue 0 (every eighth one of each kind) are dealt, longest first, to an eighth of the compute units as they become free.
// Putting the pieces together costs kMerge and the time to read the partial results.  A cut has to win 5 % of the uncut time.
// Measured, uncut -> cut (head_dim 128, 32/8 heads): 1024 queries on 32768 keys, 128 blocks of 1024 stages in two pieces each:
// forward 744 -> 472 us + 12 us to put them together (not half: 128 busy compute units hold a
// higher clock than 256); 203 queries on 1704 keys next to 611 short rows: forward 48 -> 28 + 6 us.  Chunks the estimate
// leaves alone (8192 queries on 32768 keys: 1024 equal blocks) run as before.
// Both kinds of block of a backward in one launch (N = 2, refine_bwd_split) are dealt in the order in which that launch starts them, and
// a dQ stage counts as 5/4 of a dK/dV step; what runs is the cut with the least time, no cut included.  75 chunks on which this differs from the kinds' own
// cuts with finer pieces, which ran whatever the estimate said of them: backward 6.3 % less in the mean, none more by 1 % (both counted alike 6.2
// % and one 5 % more, 3/2 4.9 %; dealt longest first whatever the kind 5.9 % and one 8 % more; without the kinds' own cuts among the candidates 5.7 %),
// 40 others 7.7 % less, two of them 3 % more:
// 483 queries on 2437 keys, 32/8 heads, 106 -> 85 us; 3823 on 9114, 8/2, 463 -> 382; 3467 on 4302, 8/8, 177 -> 146; 11561 on 11582, 32/8, 3154.
constexpr int kJointStep = 4;
constexpr int64_t kMaxCutBlocks = 1024;  // from four blocks per compute unit on they even out by themselves

namespace {
// The walks of one kind of block (query-stationary over 32-key stages, key-stationary over query tiles).
struct CutKind {
  struct Walk { int len, n0; };  // length in units (stages or tiles); n0 of a query-stationary one
  std::vector<Walk> walks;
  int inner = 1;        // blocks per walk
  int group = 0;        // > 0: key-stationary, `group` steps per tile
  int longest = 0;      // units
  bool many = false;    // kMaxCutBlocks blocks or more: none of these is cut
  bool whole = false;   // none of these is to be cut
  int cost = 1;         // of a step, in units of the estimate
  int steps_per_unit() const { return group > 0 ? group : 1; }
  int shortest() const { return group > 0 ? (2 * kMinPieceStages + group - 1) / group : kMinPieceStages; }  // units of a piece, at least
  int pieces(const Walk& w, int target) const { return group > 0 ? tile_piece_count(w.len, target) : piece_count(w.len, w.n0, target); }
  int steps(const Walk& w, int n, int k) const {
    if (group > 0) return (share_begin(w.len, n, k + 1) - share_begin(w.len, n, k)) * group;
    return (k + 1 < n ? piece_begin(w.len, n, k + 1) : w.len) - piece_begin(w.len, n, k);
  }
  void add(int len, int n0) {
    walks.push_back(Walk{len, n0});
    longest = std::max(longest, len);
    many = (int64_t)walks.size() * inner >= kMaxCutBlocks;
  }
};

// (The choice is part of every call: blocks are counted before walks are listed.)
bool many_blocks(const chunk_attn_desc* d, bool keys, int rows, int inner) {
  int64_t n = 0;
  for (int t = 0; t < d->num_segments; ++t) n += ((keys ? d->segments[t].kv_len : d->segments[t].q_len) + rows - 1) / rows;
  return n * inner >= kMaxCutBlocks;
}

CutKind key_walks(const chunk_attn_desc* d, int tile_rows, int inner) {
  CutKind k;
  k.inner = inner;
  for (int t = 0; t < d->num_segments; ++t) {
    const chunk_attn_seg& s = d->segments[t];
    for (int32_t i0 = 0; i0 < s.q_len; i0 += tile_rows) {
      const int32_t n0 = s.kv_len - s.q_len + i0 + 1;
      k.add(walk_stages(n0, std::min<int32_t>(tile_rows, s.q_len - i0)), n0);
    }
  }
  return k;
}

// Blocks of queue 0 among the `inner` ones that start at block b: those divisible by 8.
int64_t in_queue(int64_t b, int64_t inner) { return (b + inner + 7) / 8 - (b + 7) / 8; }

// The blocks of queue 0 in the order in which they start.
struct Starts {
  struct Run { int64_t cost, blocks; };  // one after the other, of equal cost
  std::vector<Run> runs;
  int64_t work = 0, longest = 0;
  void add(int64_t cost, int64_t blocks) {
    if (blocks == 0) return;
    work += cost * blocks;
    longest = std::max(longest, cost);
    if (!runs.empty() && runs.back().cost == cost) runs.back().blocks += blocks;
    else runs.push_back(Run{cost, blocks});
  }
};

// When the last block ends if they are dealt to `workers` as they become free.
int64_t deal(const Starts& starts, int workers) {
  std::vector<int64_t> heap(workers, 0);  // when they become free, the earliest first
  int64_t* const free_at = heap.data();
  int64_t last = 0;
  for (const Starts::Run& run : starts.runs) {
    int64_t n = run.blocks;
    if (n >= workers && last - free_at[0] <= run.cost) {  // none becomes free a second time before all have: each takes one block of a round
      const int64_t rounds = n / workers;
      for (int w = 0; w < workers; ++w) free_at[w] += rounds * run.cost;
      last = *std::max_element(free_at, free_at + workers);
      n -= rounds * workers;
    }
    for (; n > 0; --n) {
      const int64_t end = free_at[0] + run.cost;
      last = std::max(last, end);
      int at = 0;  // the earliest one takes the block and sinks to its place
      for (int child; (child = 2 * at + 1) < workers; at = child) {
        if (child + 1 < workers && free_at[child + 1] < free_at[child]) ++child;
        if (free_at[child] >= end) break;
        free_at[at] = free_at[child];
      }
      free_at[at] = end;
    }
  }
  return last;
}

// From so many blocks of a queue on they even out by themselves: neither listed (a list costs the host 10 ns a block) nor dealt (20), but summed.
constexpr int64_t kManyBlocks = 1024;
// (No runs: the sum is what there is to know.)
int64_t last_end(const Starts& s, int workers) { return s.runs.empty() ? s.work / workers : deal(s, workers); }
// Whether x times the end of `a` is before y times that of `b`.  (A last block starts when the others' work has been shared out at the latest, so most pairs need no dealing.)
bool ends_before(const Starts& a, int64_t x, const Starts& b, int64_t y, int workers) {
  const bool few = !a.runs.empty() && !b.runs.empty();
  if (few && x * (a.work / workers + 1 + a.longest) < y * std::max(b.work / workers, b.longest)) return true;
  if (few && x * std::max(a.work / workers, a.longest) >= y * (b.work / workers + 1 + b.longest)) return false;
  return x * last_end(a, workers) < y * last_end(b, workers);
}

// Stages of the walks of one head, none of them cut, in the order in which a launch starts and numbers their blocks: sequence by sequence (by_sequence_then_walk).
// (Numbered by the segment table, of 350 sequences of 146 tokens with four key/value heads only the first and longer key block of each would be in queue 0.)
template <class F>
void key_walks_of(const chunk_attn_seg& s, int tile_rows, F&& walk) {
  for (int32_t i0 = (s.q_len - 1) / tile_rows * tile_rows; i0 >= 0; i0 -= tile_rows)
    walk(walk_stages(s.kv_len - s.q_len + i0 + 1, std::min<int32_t>(tile_rows, s.q_len - i0)));
}
template <class F>
void key_walks_as_started(const chunk_attn_desc* d, int tile_rows, F&& walk) {
  std::vector<int> order(d->num_segments);
  std::iota(order.begin(), order.end(), 0);
  std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return d->segments[a].kv_len > d->segments[b].kv_len; });
  for (int t : order) key_walks_of(d->segments[t], tile_rows, walk);
}
// Steps of those of key blocks, which start longest first: behind each other where whole blocks of context walk all query tiles, else counted by length.
template <class F>
void tile_walks_as_started(const chunk_attn_desc* d, int keys, F&& walks) {
  const int group = d->num_q_heads / d->num_kv_heads;
  int most = 0;
  for (int t = 0; t < d->num_segments; ++t) most = std::max(most, (d->segments[t].q_len + 31) / 32);
  std::vector<int32_t> blocks(most + 1, 0);  // by query tiles
  for (int t = 0; t < d->num_segments; ++t) {
    const chunk_attn_seg& s = d->segments[t];
    const int32_t C = s.kv_len - s.q_len, n_qt = (s.q_len + 31) / 32, whole = C / keys + 1;
    blocks[n_qt] += whole;
    for (int64_t j0 = (int64_t)whole * keys; j0 < s.kv_len; j0 += keys) ++blocks[n_qt - (j0 - C) / 32];
  }
  for (int tiles = most; tiles >= 0; --tiles)
    if (blocks[tiles] > 0) walks((int64_t)tiles * group, blocks[tiles]);
}

// The blocks of both kinds, none of them cut, as one launch starts them: a dQ block costs `dq_stage` per stage and `dq_start`
// more, a dK/dV block of `keys` keys `step` per step and `start` more.
Starts joint_starts(const chunk_attn_desc* d, int tile_rows, int inner, int keys, int dq_stage, int dq_start, int step, int start) {
  const Walks q = count_walks(d, tile_rows), k = count_dkv_walks(d, keys);
  const int64_t q_blocks = q.items * inner, k_blocks = k.items * d->num_kv_heads;
  Starts s;
  if (q_blocks + k_blocks > 8 * kManyBlocks) {
    s.work = ((q.stages * dq_stage + q.items * dq_start) * inner + (k.stages * step + k.items * start) * d->num_kv_heads) / 8;
    return s;
  }
  auto add_keys = [&]() {
    int64_t block = 0;
    key_walks_as_started(d, tile_rows, [&](int64_t stages) {
      s.add(stages * dq_stage + dq_start, in_queue(block, inner));
      block += inner;
    });
  };
  auto add_tiles = [&]() {
    int64_t block = 0;
    tile_walks_as_started(d, keys, [&](int64_t steps, int64_t n) {
      s.add(steps * step + start, in_queue(block, n * d->num_kv_heads));
      block += n * d->num_kv_heads;
    });
  };
  const bool dq_first = q.longest > k.longest;  // (bwd_layout)
  if (dq_first) add_keys();
  add_tiles();
  if (!dq_first) add_keys();
  return s;
}

CutKind tile_walks(const chunk_attn_desc* d, int keys) {
  CutKind k;
  k.inner = d->num_kv_heads;
  k.group = d->num_q_heads / d->num_kv_heads;
  for (int t = 0; t < d->num_segments; ++t) {
    const chunk_attn_seg& s = d->segments[t];
    const int32_t C = s.kv_len - s.q_len, n_qt = (s.q_len + 31) / 32;
    for (int32_t j0 = 0; j0 < s.kv_len; j0 += keys) k.add(n_qt - std::max<int32_t>(0, j0 - C) / 32, 0);
  }
  return k;
}

// The cut of N kinds of block that share the compute units, one split each; at most max_parts[i] partial results of kind i.
// `first` (or null): a cut to look at besides those into equal shares.
template <int N>
void choose_cut(const CutKind (&kinds)[N], int cus, const int64_t (&max_parts)[N], KeySplit (&best)[N], const KeySplit* first = nullptr) {
  constexpr int kUnit = N > 1 ? kJointStep : 1;  // a step
  constexpr int kStart = 12 * kUnit, kPart = 6 * kUnit, kMerge = 6 * kUnit;
  constexpr int64_t kPartsPerStep = 32;  // partial results (128 KB per block) read per step
  const int workers = std::max(1, cus / 8);
  std::vector<int64_t> cost;
  int64_t total = 0;    // work of queue 0 ...
  int largest = 0;      // ... and its longest block
  bool many = false;
  auto count_pieces = [&](KeySplit (&k)[N]) {
    for (int i = 0; i < N; ++i) {
      k[i].pieces = k[i].parts = 0;
      for (const auto& w : kinds[i].walks) {
        const int n = kinds[i].pieces(w, k[i].target);
        k[i].pieces += n;
        if (n > 1) k[i].parts += n;
      }
    }
  };
  auto count_work = [&](const KeySplit (&k)[N]) {
    total = largest = 0;
    for (int i = 0; i < N; ++i) {
      const CutKind& kind = kinds[i];
      int64_t block = 0;
      for (const auto& w : kind.walks) {
        const int n = kind.pieces(w, k[i].target);
        for (int x = 0; x < n; ++x, block += kind.inner) {
          const int64_t q = in_queue(block, kind.inner);
          if (q == 0) continue;
          const int c = kind.steps(w, n, x) * kind.cost + kStart + (n > 1 ? kPart : 0);
          total += q * c;
          largest = std::max(largest, c);
        }
      }
    }
  };
  auto merge_time = [&](const KeySplit (&k)[N]) {
    int64_t parts = 0;
    for (int i = 0; i < N; ++i) parts += k[i].parts * kinds[i].inner;
    return parts > 0 ? kMerge + parts * kUnit / kPartsPerStep : 0;
  };
  auto longest_steps = [&](int i, const KeySplit (&k)[N]) {
    int most = 0;
    for (const auto& w : kinds[i].walks) {
      const int n = kinds[i].pieces(w, k[i].target);
      for (int x = 0; x < n; ++x) most = std::max(most, kinds[i].steps(w, n, x));
    }
    return most;
  };
  // (needs count_work of the same splits)
  auto estimate = [&](const KeySplit (&k)[N]) -> int64_t {
    if (many) return std::max<int64_t>(total / workers, largest) + merge_time(k);  // many small blocks fill every gap
    Starts starts;
    const bool swap = N > 1 && longest_steps(0, k) <= longest_steps(N - 1, k);  // the kind with the longer walks starts first (bwd_layout)
    for (int j = 0; j < N; ++j) {
      const int i = swap ? N - 1 - j : j;
      const CutKind& kind = kinds[i];
      int64_t block = 0;
      cost.clear();
      for (const auto& w : kind.walks) {
        const int n = kind.pieces(w, k[i].target);
        for (int x = 0; x < n; ++x, block += kind.inner)
          cost.insert(cost.end(), in_queue(block, kind.inner), kind.steps(w, n, x) * kind.cost + kStart + (n > 1 ? kPart : 0));
      }
      std::sort(cost.begin(), cost.end(), [](int64_t a, int64_t b) { return a > b; });
      for (int64_t c : cost) starts.add(c, 1);
    }
    return deal(starts, workers) + merge_time(k);
  };
  int longest = 0, shortest = 0x7fffffff;  // steps
  for (int i = 0; i < N; ++i) {
    best[i] = KeySplit{};
    many |= kinds[i].many;
    if (kinds[i].many || kinds[i].whole) continue;
    longest = std::max(longest, kinds[i].longest * kinds[i].steps_per_unit());
    shortest = std::min(shortest, kinds[i].shortest() * kinds[i].steps_per_unit());
  }
  if (longest == 0) return;  // nothing that may be cut
  count_pieces(best);
  count_work(best);
  int64_t best_time = estimate(best);
  best_time -= best_time / 20;
  if (total / workers >= best_time) return;  // as even as it can get: pieces only add to the work
  // The choice is part of every call, so a candidate that cannot win is not followed further: one with too many partial
  // results, or whose work shared evenly, or longest block alone, already takes as long as the best so far.
  bool found = false;
  auto consider = [&](KeySplit (&k)[N]) {  // (pieces counted)
    count_work(k);
    if (std::max<int64_t>(total / workers, largest) + merge_time(k) >= best_time) return;
    const int64_t time = estimate(k);
    if (time >= best_time) return;
    std::copy(k, k + N, best);
    best_time = time;
    found = true;
  };
  if (first) {
    KeySplit k[N];
    std::copy(first, first + N, k);
    count_pieces(k);
    consider(k);
  }
  for (int n = 2; n <= 16 && longest / n >= shortest; ++n) {
    KeySplit k[N];
    for (int i = 0; i < N; ++i) {
      const int unit = kinds[i].steps_per_unit(), target = ((longest + n - 1) / n + unit - 1) / unit;
      if (!kinds[i].many && !kinds[i].whole && kinds[i].longest > target) k[i].target = std::max(target, kinds[i].shortest());
    }
    count_pieces(k);
    int64_t blocks = 0, parts = 0;
    bool fits = true;
    for (int i = 0; i < N; ++i) {
      if (!kinds[i].many) blocks = std::max(blocks, k[i].pieces * kinds[i].inner);
      parts += k[i].parts;
      fits &= k[i].parts <= max_parts[i];
    }
    if (blocks > 2 * kMaxCutBlocks) break;
    if (parts == 0 || !fits) continue;
    consider(k);
  }
  // a kind whose cut brings nothing stays whole
  if (N > 1 && found) {
    for (int i = 0; i < N; ++i) {
      if (best[i].parts == 0) continue;
      KeySplit k[N];
      std::copy(best, best + N, k);
      k[i].target = 0;
      count_pieces(k);
      count_work(k);
      if (estimate(k) <= best_time + best_time / 50) std::copy(k, k + N, best);
    }
  }
  for (KeySplit& k : best)
    if (k.parts == 0) k.target = 0;
}
}  // namespace

constexpr int kLongSharedWalk = 40;
constexpr int kMaxSharedHeads = 4096;  // block counts and byte offsets inside a tile stay in 32 bits (no chunk of as many heads is small)

// Times (us) of the two kinds of forward.  Least squares in the logarithm over 8500 drawn chunks of up to 104 tiles of 32 rows (1 - 3300 queries, up to
// 6 contexts of up to 20000 keys, 1 - 128 query and 1 - 64 key/value heads), each measured with every choice, 5000 of them on the tensors of the call
// before (in the caches where they fit) and 3500 on tensors that come from memory.  Off by 5 - 10 % (root mean square; the other kernels by 7).  A
// stage from memory costs this kernel more than the other ones (at 96 and 128 one head to a workgroup has room for a single slot per wave: its
// copies' latency shows), so there are two sets, and the choice has to be ahead by both.  A single set for tensors in the caches, without the
// rounds of workgroups and the pieces of cut walks, was up to 1.7 times slower than the other kernel where few queries meet thousands of keys of many
// key/value heads (13 queries on 14478 keys, 64/64, head_dim 96: 104 -> 172; 4 on 7246, 128/16, 128, from memory: 49 -> 80).  Of 10000 chosen
// chunks of other draws 17 are slower by more than 2 %, by 16 % at most (71 heads on one key/value head), of 8500 from memory 41, by 21 % at most (258
// queries on 4180 keys, 32/8, 128).  All chunks together, by head_dim 64, 96 and 128, 1.64, 1.51 and 1.56 times as fast as without the kernel (from
// memory 1.36, 1.36 and 1.38), where the best choice would be 1.66, 1.59 and 1.66 (1.37, 1.40 and 1.42).
// Examples, other kernel -> one, two, four heads: head_dim 64, 1024 tokens, 8/8 heads, 16.9 -> 7.9; four sequences of 512, 256, 128 and 128,
// 8/8, 10.6 -> 6.0, 32/8, 11.1 -> 15.8, 9.3, 10.5; 100 queries on 10100 keys, 32/8, 124 -> 40, 62, 110; head_dim 128, 203 queries on 1704 keys with
// 611 packed tokens, 32/8, 30.1 -> 26.1, 21.6, 31.7; eight sequences of 128, 32/8, 14.4 -> 18.1, 12.8, 9.7; 200 queries on 20200 keys, 32/8,
// 90 -> 123, 192, 293 (walks cut over the whole chip).
struct SharedCost {  // the larger of what the longest walk and what all workgroups take; rounds: workgroups over those on the chip at a time, rounded up
  double first, step, all_steps, workgroup, longest, mb, round;
  int slots;  // workgroups on the chip at a time
  double us(double most, double steps, double workgroups, double kv_mb) const {
    return first + std::max(step * most, (all_steps * steps + workgroup * workgroups) / slots + longest * most) + mb * kv_mb + round * std::ceil(workgroups / slots);
  }
};
// [tensors in the caches, from memory][one, two, four heads].  (At 96 and 128 the step of one head from memory is 1.1 times the mean one.)
constexpr SharedCost kShared64[2][3] = {
    {{1.72, 0.771, 1.01, 0.23, 0.033, 0.083, 1.75, 256}, {2.83, 0.739, 1.24, 1.89, 0.315, 0.017, 0.75, 512}, {3.14, 0.642, 0.953, 2.59, 0.394, 0.047, 1.09, 512}},
    {{4.79, 1.12, 1.01, 0.59, 0.18, 0.44, 1.72, 256}, {5.62, 0.993, 1.20, 2.50, 0.29, 0.62, 0.90, 512}, {6.86, 0.638, 0.92, 4.15, 0.43, 0.046, 0.76, 512}}};
constexpr SharedCost kShared96[2][3] = {
    {{2.23, 1.14, 1.57, 0.60, 0.035, 0.126, 1.70, 256}, {2.80, 1.04, 1.17, 1.46, 0.20, 0.025, 1.18, 256}, {3.95, 0.81, 0.914, 2.90, 0.12, 0.023, 1.0, 256}},
    {{4.88, 2.06, 1.54, 0.95, 0.515, 0.30, 1.66, 256}, {5.77, 1.38, 1.21, 2.07, 0.29, 0.43, 1.01, 256}, {7.41, 0.807, 0.87, 3.78, 0.24, 0.061, 1.14, 256}}};
constexpr SharedCost kShared128[2][3] = {
    {{1.94, 1.19, 1.53, 0.51, 0.07, 0.093, 2.08, 256}, {2.74, 1.15, 1.28, 1.43, 0.28, 0.029, 1.63, 256}, {4.32, 0.954, 1.105, 3.21, 0.16, 0.011, 1.19, 256}},
    {{4.65, 2.30, 1.53, 1.05, 0.68, 0.23, 1.75, 256}, {5.78, 1.50, 1.31, 2.03, 0.40, 0.33, 1.48, 256}, {7.94, 0.948, 0.935, 4.43, 0.45, 0.024, 1.18, 256}}};
// The other kernels: that of 64, a workgroup per block, and the pipelined one of 96 and 128, whose walks may be cut into pieces.
struct PlainFwdCost {
  double first, walk, all, block, longest, mb;
  double us(const Walks& w, double inner, double kv_mb) const {
    const double per_cu = inner / 256;
    return first + std::max(walk * w.longest, (all * w.stages + block * w.items) * per_cu + longest * w.longest) + mb * kv_mb;
  }
};
struct PipeFwdCost {
  double first, piece, all, round, block, cut, part, mb;
  double us(const Walks& w, const KeySplit& split, double inner, double kv_mb) const {
    const double per_cu = inner / 256, blocks = (split.target > 0 ? split.pieces : w.items) * per_cu;
    const double longest = (double)(split.target > 0 ? std::min<int64_t>(split.target, w.longest) : w.longest);
    return first + std::max(piece * longest, all * w.stages * per_cu) + round * std::ceil(blocks) + block * blocks +
           (split.target > 0 ? cut + part * split.parts * per_cu : 0.0) + mb * kv_mb;
  }
};
constexpr PlainFwdCost kOther64[2] = {{3.98, 0.368, 0.186, 1.10, 0.319, 0.0}, {7.44, 0.382, 0.182, 1.74, 0.305, 0.195}};
constexpr PipeFwdCost kOther96[2] = {{0.66, 0.618, 0.709, 7.84, 2.80, 6.09, 2.35, 0.021}, {5.71, 0.606, 0.708, 7.39, 4.23, 5.97, 0.0, 0.092}};
constexpr PipeFwdCost kOther128[2] = {{1.52, 0.687, 0.796, 7.87, 3.55, 7.56, 1.62, 0.037}, {6.04, 0.673, 0.788, 8.05, 4.90, 7.15, 0.0, 0.108}};
constexpr double kAheadFwd = 0.97;  // share of the other kernel's time that is asked for

int choose_shared_heads(const chunk_attn_desc* d, const Walks& other, int inner, bool pipelined, const KeySplit& split) {
  if (d->head_dim > 128 || (d->head_dim == 64 && pipelined) || d->num_q_heads > kMaxSharedHeads) return 0;
  // (long walks that are not cut: mostly enough blocks for the chip, and the pipelined kernel's steps are cheaper.  Of 247 drawn chunks 121 were slower
  // with this kernel by more than 2 %, up to 2.8 times; 100 would gain more than 15 %, which the line gives away: few blocks that no cut takes)
  if (d->head_dim != 64 && split.target == 0 && other.longest > kLongSharedWalk) return 0;
  int64_t items = 0;
  for (int t = 0; t < d->num_segments; ++t) {
    items += (d->segments[t].q_len + 31) / 32;
    if (items > kMaxSharedItems) return 0;
  }
  int64_t keys = 0;
  for (int t = 0; t < d->num_segments; ++t) keys += d->segments[t].kv_len;
  const double kv_mb = (double)keys * d->num_kv_heads * d->head_dim * 4e-6;
  double limit[2];  // what the shared kernel may take
  for (int m = 0; m < 2; ++m)
    limit[m] = kAheadFwd * (d->head_dim == 64 ? kOther64[m].us(other, inner, kv_mb) : (d->head_dim == 96 ? kOther96 : kOther128)[m].us(other, split, inner, kv_mb));
  const SharedCost(&costs)[2][3] = d->head_dim == 64 ? kShared64 : d->head_dim == 96 ? kShared96 : kShared128;
  const int group = d->num_q_heads / d->num_kv_heads;
  int best = 0;
  double best_share = 1.0;
  for (int x = 0; x < 3; ++x) {
    const int heads = 1 << x, splits = kSharedWaves / heads;
    if (group % heads != 0) break;
    int64_t steps = 0, most = 0;
    for (int t = 0; t < d->num_segments; ++t) {
      const chunk_attn_seg& s = d->segments[t];
      for (int i0 = 0; i0 < s.q_len; i0 += 32) {
        const int64_t n = (walk_stages(s.kv_len - s.q_len + i0 + 1, std::min(32, s.q_len - i0)) + splits - 1) / splits;
        steps += n;
        most = std::max(most, n);
      }
    }
    const double wgs = (double)(d->num_q_heads / heads);
    auto share = [&](int m) { return costs[m][x].us((double)most, steps * wgs, items * wgs, kv_mb) / limit[m]; };
    const double cached = share(0), memory = share(1);
    if (cached < 1.0 && memory < 1.0 && cached * memory < best_share) {
      best_share = cached * memory;
      best = heads;
    }
  }
  return best;
}

// The same for the backward, least squares over 5000 drawn chunks on the tensors of the call before.  Off by 5 - 8 % (root mean square), the other
// kernels by 7 - 9.  (From memory this kernel gains on the other ones, so one set is enough.)  An estimate from 1290 chunks that knew neither rounds nor
// the pieces of cut walks, off by 8 - 19 % for the other kernels, was slower by more than 2 % in 122 of 13000 chosen chunks of other draws, by up to 38 % (17
// queries on 1551 keys in two sequences, 128/16 heads, head_dim 128: 35.5 -> 48.9; 7 on 2747, 64/8: 33 -> 40; 38 on 2460, 32/8, 96: 31.1 -> 34.0).  With
// this one and the shares asked for, 9 of 11000 chosen chunks of other draws are, by 14 % at most, 2 of 5700 from memory, by 3 %.  All chunks together,
// by head_dim 64, 96 and 128, 1.65, 1.34 and 1.38 times as fast as without the kernel (from memory 1.58, 1.35 and 1.35), where the best choice would be
// 1.76, 1.51 and 1.56 (1.67, 1.49 and 1.51): most of the difference is in the chunks that choose_shared_waves refuses outright.
// Examples, other kernels -> this one: head_dim 64, 8/8 heads, 64 tokens, 8.7 -> 5.3, sequences of 256, 512, 128 and 128, 19.5 -> 10.4, 1024 tokens, 29.4 ->
// 15.7; 100 queries on 10100 keys, 32/8, 175 -> 72; head_dim 128, 8/8, 500 tokens, 33.4 -> 14.7, 1000, 46.7 -> 27.8, 100 queries on 1100 keys, 45 -> 17.
struct SharedBwdCost {
  double first, dq_step, dkv_step, all_dq, all_dkv, workgroup, longest, round, mb;
  int waves, slots;
  double us(double dq_most, double dkv_most, double dq_all, double dkv_all, double blocks, double kv_mb) const {
    return first + std::max({dq_step * dq_most, dkv_step * dkv_most,
                             (all_dq * dq_all + all_dkv * dkv_all + workgroup * blocks) / slots + longest * std::max(dq_most, dkv_most)}) +
           round * std::ceil(blocks / slots) + mb * kv_mb;
  }
};
constexpr SharedBwdCost kSharedBwd64[2] = {{4.13, 0.565, 1.068, 1.94, 0.592, 2.08, 0.087, 0.443, 0.168, 4, 512}, {4.07, 0.641, 1.488, 2.51, 0.277, 1.03, 0.152, 0.402, 0.818, 8, 256}};
constexpr SharedBwdCost kSharedBwd96 = {5.06, 0.881, 1.664, 1.433, 1.469, 2.65, 0.137, 0.955, 0.067, 4, 256};
constexpr SharedBwdCost kSharedBwd128 = {5.53, 0.969, 1.762, 1.754, 1.415, 2.87, 0.13, 0.922, 0.093, 4, 256};
struct OtherBwdCost {
  double first, dq_piece, dkv_piece, all_dq, all_dkv, block, round, cut, part, mb;
};
constexpr OtherBwdCost kOtherBwd64 = {5.99, 0.487, 0.728, 0.32, 0.877, 1.80, 0.878, 2.24, 15.3, 0.156};
constexpr OtherBwdCost kOtherBwd96 = {8.69, 0.634, 0.835, 0.493, 0.982, 6.37, 6.23, 4.35, 17.4, 0.223};
constexpr OtherBwdCost kOtherBwd128 = {9.44, 0.723, 0.94, 0.841, 1.04, 6.37, 7.24, 5.33, 15.6, 0.213};
constexpr double kAheadBwd64 = 0.90, kAheadBwd96 = 0.82, kAheadBwd128 = 0.85;  // shares of the other kernels' time that are asked for

bool shared_backward_fits(const chunk_attn_desc* d) {
  if (d->num_segments > kMaxShareSegs || d->num_q_heads > kMaxSharedHeads) return false;
  int64_t items = 0;
  for (int t = 0; t < d->num_segments; ++t) items += (d->segments[t].q_len + 31) / 32 + ((int64_t)d->segments[t].kv_len + 31) / 32;
  return items <= kMaxShareItems;
}

int choose_shared_waves(const chunk_attn_desc* d, int head_dim, const Walks& dq, int inner, const Walks& dkv, const KeySplit& dq_split, const KeySplit& dkv_split) {
  const bool dq_cut = dq_split.target > 0, dkv_cut = dkv_split.target > 0, cut = dq_cut || dkv_cut;
  // (long dK/dV walks are cut evenly already; dQ walks are not.  Of 393 drawn chunks 120 were slower with this kernel by more than 2 %, up to 3.1
  // times, and 190 would gain more than 15 %, up to 2.6 times, which the line gives away)
  if (head_dim == 64 && cut && dq.longest <= dkv.longest && dkv.longest > 32) return 0;
  // (as in the forward.  Of 647 drawn chunks 183 were slower by more than 2 %, up to 2.2 times; 439 would gain more than 15 %, up to 3.2 times, which the
  // line gives away: few queries on a long context, whose dQ walks find no room for partial results, 10 on 14018 keys, 8/8 heads, head_dim 128,
  // 377 us where this kernel takes 118)
  if (head_dim != 64 && !cut && dq.longest > kLongSharedWalk) return 0;
  const int group = d->num_q_heads / d->num_kv_heads;
  int64_t keys = 0;
  for (int t = 0; t < d->num_segments; ++t) keys += d->segments[t].kv_len;
  const double kv_mb = (double)keys * d->num_kv_heads * head_dim * 4e-6;
  const OtherBwdCost& o = head_dim == 64 ? kOtherBwd64 : head_dim == 96 ? kOtherBwd96 : kOtherBwd128;
  const double dq_piece = (double)(dq_cut ? std::min<int64_t>(dq_split.target, dq.longest) : dq.longest);
  const double dkv_piece = (double)(dkv_cut ? std::min<int64_t>((int64_t)dkv_split.target * group, dkv.longest) : dkv.longest);
  const double blocks = (double)((dq_cut ? dq_split.pieces : dq.items) * inner + (dkv_cut ? dkv_split.pieces : dkv.items) * d->num_kv_heads) / 256;
  const double parts = (double)((dq_cut ? dq_split.parts : 0) * inner + (dkv_cut ? dkv_split.parts : 0) * d->num_kv_heads) / 256;
  const double other = o.first +
                       std::max({o.dq_piece * dq_piece, o.dkv_piece * dkv_piece,
                                 (o.all_dq * dq.stages * inner + o.all_dkv * dkv.stages * d->num_kv_heads) / 256 + o.block * blocks}) +
                       o.round * std::ceil(blocks) + (cut ? o.cut : 0.0) + o.part * parts + o.mb * kv_mb;
  int best = 0;
  double best_us = (head_dim == 64 ? kAheadBwd64 : head_dim == 96 ? kAheadBwd96 : kAheadBwd128) * other;
  for (int x = 0; x < (head_dim == 64 ? 2 : 1); ++x) {
    const SharedBwdCost& c = head_dim == 64 ? kSharedBwd64[x] : head_dim == 96 ? kSharedBwd96 : kSharedBwd128;
    int64_t dq_most = 0, dkv_most = 0, dq_all = 0, dkv_all = 0, dq_items = 0, dkv_items = 0;
    auto add = [&](int64_t steps, int64_t& items_of_kind, int64_t& most, int64_t& all) {
      ++items_of_kind;
      steps = (steps + c.waves - 1) / c.waves;
      most = std::max(most, steps);
      all += steps;
    };
    for (int t = 0; t < d->num_segments; ++t) {
      const chunk_attn_seg& s = d->segments[t];
      const int32_t C = s.kv_len - s.q_len, n_qt = (s.q_len + 31) / 32;
      for (int32_t i0 = 0; i0 < s.q_len; i0 += 32) add(walk_stages(C + i0 + 1, std::min(32, s.q_len - i0)), dq_items, dq_most, dq_all);
      for (int32_t j0 = 0; j0 < s.kv_len; j0 += 32) add((int64_t)(n_qt - std::max(0, j0 - C) / 32) * group, dkv_items, dkv_most, dkv_all);
    }
    const double us = c.us((double)dq_most, (double)dkv_most, (double)dq_all * d->num_q_heads, (double)dkv_all * d->num_kv_heads,
                           (double)(dq_items * d->num_q_heads + dkv_items * d->num_kv_heads), kv_mb);
    if (us < best_us) {
      best_us = us;
      best = c.waves;
    }
  }
  return best;
}

KeySplit choose_key_split(const chunk_attn_desc* d, int tile_rows, int inner, int cus, int64_t max_parts) {
  if (many_blocks(d, false, tile_rows, inner)) return KeySplit{};
  const CutKind kinds[1] = {key_walks(d, tile_rows, inner)};
  KeySplit best[1];
  choose_cut<1>(kinds, cus, {max_parts}, best);
  return best[0];
}

KeySplit choose_tile_split(const chunk_attn_desc* d, int keys, int cus, int64_t max_parts) {
  if (many_blocks(d, true, keys, d->num_kv_heads)) return KeySplit{};
  const CutKind kinds[1] = {tile_walks(d, keys)};
  KeySplit best[1];
  choose_cut<1>(kinds, cus, {max_parts}, best);
  return best[0];
}

void refine_bwd_split(const chunk_attn_desc* d, int tile_rows, int inner, int keys, int cus, int64_t max_parts, KeySplit* dq, KeySplit* dkv) {
  if (dq->target == 0 && dkv->target == 0) return;
  CutKind kinds[2] = {key_walks(d, tile_rows, inner), tile_walks(d, keys)};
  kinds[0].whole = dq->target == 0;
  kinds[1].whole = dkv->target == 0;
  kinds[0].cost = 5;  // 48 MFMAs per wave and stage, against 32 per step of dK/dV: not 3 : 2, as other costs of a step are alike
  kinds[1].cost = kJointStep;
  const KeySplit alone[2] = {*dq, *dkv};
  KeySplit best[2];
  choose_cut<2>(kinds, cus, {max_parts / inner, max_parts / d->num_kv_heads}, best, alone);
  *dq = best[0];
  *dkv = best[1];
}

// The estimate of refine_bwd_split for uncut walks, with the dK/dV blocks of either size: a step of 256 keys counts as 8/5 of one of 128 (1.61 by its cycles), the start and end of
// either as ten steps of 128 and of a dQ block as twelve, and 256 keys have to be ahead by a twentieth, for what the estimate cannot tell apart keeps the blocks of 128 (where dQ blocks start first, just
// ahead: the ends of few dK/dV blocks behind them come out too late).  Of 999 drawn chunks of 60 us and more (backward, 128 and 96, up to 65536 keys, 1 - 8 query heads to a key/value head, two
// thirds of them of many short sequences) it picks 634, of which seven are slower by more than 1.5 % (2.9 at most: 277 sequences, 63653 tokens, 64/8 heads, 2902 us); all 999 take 4.6 % less in the
// mean.  (Without the margin, and 16 steps for the start of 256 keys, 18 of 924 are slower, by 34 % at most.)
// 14147 queries on 14216 keys, 32/8 heads, 4718 -> 4283 us; 4977 on 38367, 64/8, 16275 -> 15116; 3193 on 8192, 32/8, 1116 -> 1044; eight sequences of 300 tokens, 64/64, 216 -> 204;
// what stays: 5251 causal tokens, 32/8, 687 (blocks of 256 keys: 931), 4596, 40/8, 680 (982), 6403 on 10177, 28/4, 1884 (2032), 129 sequences of 222 tokens, 40/8, 834 (868).
bool tall_pays(const chunk_attn_desc* d, int tile_rows, int inner, int keys, int cus) {
  constexpr int kStep = 20, kDqStage = 25, kTallStep = 32, kDqStart = 12 * kStep, kStart = 10 * kStep;
  const bool dq_first = count_walks(d, tile_rows).longest > count_dkv_walks(d, keys).longest;  // (bwd_layout)
  return ends_before(joint_starts(d, tile_rows, inner, kTallKeys, kDqStage, kDqStart, kTallStep, kStart), 20,
                     joint_starts(d, tile_rows, inner, keys, kDqStage, kDqStart, kStep, kStart), dq_first ? 20 : 19, std::max(1, cus / 8));
}

// Pipelined from two blocks of `keys` per CU and 14 steps each on average on, unless most of the larger blocks' second halves are empty (sequences of up to 64 keys: 331 of
// 51 tokens, 28/4 heads, unpipelined / pipelined 649 / 801 us; 278 of 70 934 / 784).  Below that chunks whose dQ walks are of 8 stages or more on average are decided by
// estimates in us: the pipelined blocks of both kinds dealt as in tall_pays; the unpipelined ones, whose walks may be cut
// and so know no longest one, by their number and steps.  Least squares in the relative error over 1140 drawn chunks of 60 us and more (up to 65536 keys, 1 - 8 query heads to a
// key/value head, two thirds of them of many short sequences), each run both ways; off by 7 and 10 % (root mean square), so that the pipelined ones have to be ahead by 5.  Of the 1140 it
// picks 755, of which three are slower by more than 1.5 % than without these blocks (3.0 at most: 2112 causal tokens, 8/8, 106 us); all take 11.0 % less in the mean, with
// the better of the two for each 13.1.  Of the walks of 5 to 8 stages it would pick 74, 3 to 18 % faster; those that take less than 60 us (ten sequences of 200 tokens, 4/4 heads), which were not
// measured, look the same to it, and all of them keep the unpipelined blocks.  Unpipelined / pipelined: 2668 causal tokens, 8/8 heads, 184 / 148 us; 1428 queries on
// 3445 keys, 32/8, 578 / 407; 10770 causal, 28/4, 7202 / 4677; 7307, 32/8, 3571 / 2456; what stays: 4335, 8/2, 386 / 655; 899, 64/8, 172 / 298.
bool wide_pays(const chunk_attn_desc* d, int tile_rows, int inner, int keys, int cus) {
  const Walks w = count_dkv_walks(d, keys);
  if (w.items * d->num_kv_heads >= 2 * cus && w.stages >= 14 * w.items && 4 * count_tiles(d, true, kWideKeys) <= 3 * w.items) return true;
  const Walks wq = count_walks(d, tile_rows);
  if (wq.stages < 8 * wq.items) return false;
  constexpr int kUs = 20, kDqStage = 24, kDqStart = 18 * kUs, kStep = 26, kStart = 15 * kUs;
  const double pipelined = 4.7 + 1.035 / kUs * last_end(joint_starts(d, tile_rows, inner, kWideKeys, kDqStage, kDqStart, kStep, kStart), std::max(1, cus / 8));
  const double per_cu = 1.0 / cus, dq_all = std::max((double)wq.stages * inner * per_cu, (double)wq.longest);
  const double other = 20.7 + 0.138 * dq_all + (16.5 * wq.items * inner + (2.09 * w.stages + 10.0 * w.items) * d->num_kv_heads) * per_cu;
  return pipelined < 0.95 * other;
}

// Blocks dealt as in tall_pays, in a fifth of a stage of 32 rows per wave, whose start and end take as long as seven of them; a stage of 64 rows counts as 7/5, its start and end as
// 15 stages.  Either kernel runs its stages in pairs, with one more for the last product.  Where a workgroup takes one head (an odd number of heads to a key/value head: 256 rows to a block of 64 per
// wave), some wave masks keys in most stages of a short walk, and 64 rows have to take a twenty-fifth less work and end sooner; elsewhere no more work, and a twenty-fifth
// later by the estimate is soon enough from two blocks of 64 rows per compute unit on.  With a few more blocks than compute units the end hangs on their order: ahead by a twentieth;
// with no more, they all start at once, and the end alone decides (up to 1.06 of the other's: of 42 such chunks those below are faster by 2 - 30 %, those above slower but for one).  Of 840 drawn chunks (up to 65536 keys, 1 - 8 query
// heads to a key/value head, two thirds of them of many short sequences) it picks 394, of which one is slower by more than 1.5 % (1.9: eleven sequences
// of 333 tokens, 32/16 heads, 80 us); all 840 take 5.3 % less in the mean, with the better of the two for each 5.5.  (Without the pairs, and by the end alone: 31 are slower, by 9 % at most.)  32 / 64 rows
// per wave: 8192 queries on 32768 keys, 32/8 heads, 7329 / 5658 us, 4096 causal tokens 302 / 242; what stays: 2668 causal tokens, 8/8, 85 / 115, 62 sequences of 241 tokens, 28/4, 235 /
// 250, eight of 1520, 8/8, 126 / 134, eleven of 701, 8/8, 64 / 71.
bool fwd_tall_pays(const chunk_attn_desc* d, int tile_rows, int inner, int cus) {
  const Walks w32 = count_walks(d, tile_rows), w64 = count_walks(d, 2 * tile_rows);
  if (w32.items * inner <= cus) return false;  // (all blocks run at once, and short ones end sooner)
  auto starts = [&](int rows, int64_t items, int stage, int start, int64_t* work) {
    Starts s;
    *work = 0;
    auto cost = [&](int stages) { return (int64_t)((stages & ~1) + 2) * stage + start; };
    for (int t = 0; t < d->num_segments; ++t) key_walks_of(d->segments[t], rows, [&](int stages) { *work += cost(stages); });
    s.work = *work * inner / 8;
    if (items * inner > 8 * kManyBlocks) return s;
    s.work = 0;
    int64_t block = 0;
    key_walks_as_started(d, rows, [&](int stages) {
      s.add(cost(stages), in_queue(block, inner));
      block += inner;
    });
    return s;
  };
  int64_t work32, work64;
  const Starts rows32 = starts(tile_rows, w32.items, 5, 35, &work32), rows64 = starts(2 * tile_rows, w64.items, 7, 75, &work64);
  const int64_t blocks = w64.items * inner;
  const int workers = std::max(1, cus / 8);
  if (blocks <= cus) return ends_before(rows64, 100, rows32, 106, workers);
  const bool one_head = tile_rows >= 128;
  return 100 * work64 < (one_head ? 96 : 100) * work32 &&
         ends_before(rows64, 100, rows32, 4 * blocks <= 5 * cus ? 95 : one_head || blocks <= 2 * cus ? 100 : 104, workers);
}

std::vector<DkvItem> cut_items(const std::vector<DkvItem>& wholes, int target, std::vector<DkvItem>* cut) {
  std::vector<DkvItem> items;
  int32_t part = 0;
  for (const DkvItem& whole : wholes) {
    const int tiles = whole.n_qt - whole.qt_first, n = tile_piece_count(tiles, target);
    if (n > 1) {
      cut->push_back(whole);
      cut->back().part = part;
      cut->back().pieces = n;
    }
    for (int k = 0; k < n; ++k) {
      DkvItem it = whole;
      it.qt_first = whole.qt_first + share_begin(tiles, n, k);
      it.n_qt = whole.qt_first + share_begin(tiles, n, k + 1);
      it.part = n > 1 ? part++ : -1;
      items.push_back(it);
    }
  }
  std::stable_sort(items.begin(), items.end(), [](const DkvItem& a, const DkvItem& b) {
    const int la = a.n_qt - a.qt_first, lb = b.n_qt - b.qt_first;
    return la != lb ? la > lb : a.q_row_seg != b.q_row_seg ? a.q_row_seg < b.q_row_seg : a.qt_first < b.qt_first;
  });
  return items;
}

std::vector<FwdItem> cut_items(std::vector<FwdItem>& wholes, int target) {
  std::vector<FwdItem> items;
  int32_t part = 0;
  for (FwdItem& whole : wholes) {
    const int stages = walk_stages(whole.n0, whole.q_rows), n = piece_count(stages, whole.n0, target);
    whole.pieces = n;
    whole.part = n > 1 ? part : -1;
    for (int k = 0; k < n; ++k) {
      const int b = piece_begin(stages, n, k) * kStageKeys;
      FwdItem it = whole;
      it.kv_row0 += b;
      it.n0 -= b;
      it.keys = (k + 1 < n ? piece_begin(stages, n, k + 1) * kStageKeys : whole.keys) - b;
      it.part = n > 1 ? part++ : -1;
      items.push_back(it);
    }
  }
  return items;
}

std::vector<DqItem> cut_items(const std::vector<DqItem>& wholes, int target, std::vector<DqItem>* cut) {
  std::vector<DqItem> items;
  int32_t part = 0;
  for (const DqItem& whole : wholes) {
    const int stages = walk_stages(whole.n0, whole.q_rows), n = piece_count(stages, whole.n0, target);
    if (n > 1) {
      cut->push_back(whole);
      cut->back().part = part;
      cut->back().pieces = n;
    }
    for (int k = 0; k < n; ++k) {
      const int b = piece_begin(stages, n, k) * kStageKeys;
      DqItem it = whole;
      it.kv_row0 += b;
      it.n0 -= b;
      it.keys = (k + 1 < n ? piece_begin(stages, n, k + 1) * kStageKeys : whole.keys) - b;
      it.part = n > 1 ? part++ : -1;
      items.push_back(it);
    }
  }
  return items;
}

// Order and walk directions of one sequence's key blocks, given in key order (= longest walk first), when `width` of
// them run side by side and read the same stream of query rows through one L2.  Blocks that start together stay
// together only if they start at the same row; blocks of unequal length end at different times.  So:
//   * blocks that every query sees come first, walking upwards: equal walks, started together at the first row;
//   * of the others (walks that begin at the block's diagonal and all end at the last row) the longest `width` walk
//     DOWN from the last row, started together; as each ends, at its diagonal, its workgroup takes the partner that
//     makes the pair's length the same for all -- the shortest remaining walks, longest of them first, walking UP:
//     a block that ends its descent at row r after time T - r is followed by one that starts its ascent near the row
//     where the others are by then; all of them arrive at the last row together, and the next `width` longest descend;
//   * the shortest quarter is kept for the end, longest first, walking upwards: small items for the workgroups to
//     even out what their unequal speeds have left.
// The result holds indices into the input order; reverse[i] is the direction of input block i.
void side_by_side_order(const std::vector<DkvItem>& blocks, int width, std::vector<int>& order, std::vector<char>& reverse) {
  const int n = (int)blocks.size();
  order.clear();
  reverse.assign(n, 0);
  int lo = 0;
  while (lo < n && blocks[lo].qt_first == 0 && blocks[lo].j0 + blocks[lo].kv_rows <= blocks[lo].ctx) order.push_back(lo++);
  int hi = n - (n - lo) / 4;
  const int tail = hi;
  while (lo < hi) {
    const int m = hi - lo;
    const int down = m >= 2 * width ? width : (m + 1) / 2, up = std::min(down, m - down);
    for (int i = 0; i < down; ++i) {
      order.push_back(lo + i);
      reverse[lo + i] = 1;
    }
    for (int i = 0; i < up; ++i) order.push_back(hi - up + i);
    lo += down;
    hi -= up;
  }
  for (int i = tail; i < n; ++i) order.push_back(i);
}

std::vector<DkvItem> plan_dkv(const chunk_attn_desc* d, int keys, int side_by_side) {
  std::vector<DkvItem> items;
  int32_t q_tile0 = 0;
  for (int t = 0; t < d->num_segments; ++t) {
    const chunk_attn_seg& s = d->segments[t];
    const int32_t C = s.kv_len - s.q_len;
    const int32_t n_qt = (s.q_len + 31) / 32;
    for (int32_t j0 = 0; j0 < s.kv_len; j0 += keys) {
      DkvItem it{};
      it.kv_row0 = s.kv_start + j0;
      it.kv_rows = std::min<int32_t>(keys, s.kv_len - j0);
      it.j0 = j0;
      it.ctx = C;
      it.q_row_seg = s.q_start;
      it.q_len = s.q_len;
      it.qt_first = std::max<int32_t>(0, j0 - C) / 32;  // query i sees key j0 iff i >= j0 - C
      it.n_qt = n_qt;
      it.q_tile0 = q_tile0;
      it.part = -1;
      items.push_back(it);
    }
    q_tile0 += (s.q_len + 63) / 64;
  }
  // sequence by sequence, longest first; the key blocks of a sequence in key order, which is longest walk first (see
  // by_sequence_then_walk)
  std::stable_sort(items.begin(), items.end(), [](const DkvItem& a, const DkvItem& b) { return a.n_qt > b.n_qt; });
  if (side_by_side <= 0) return items;
  std::vector<DkvItem> out;
  out.reserve(items.size());
  std::vector<DkvItem> seq;
  std::vector<int> order;
  std::vector<char> reverse;
  for (size_t i = 0; i < items.size();) {
    size_t e = i;
    while (e < items.size() && items[e].q_row_seg == items[i].q_row_seg && items[e].kv_row0 - items[e].j0 == items[i].kv_row0 - items[i].j0) ++e;
    seq.assign(items.begin() + i, items.begin() + e);
    side_by_side_order(seq, side_by_side, order, reverse);
    for (int k : order) {
      out.push_back(seq[k]);
      out.back().reverse = reverse[k];
    }
    i = e;
  }
  return out;
}

int fused_num_bufs(const chunk_attn_desc* d, int keys) {
  int most = 0;
  for (int t = 0; t < d->num_segments; ++t) most = std::max(most, (d->segments[t].kv_len + keys - 1) / keys);
  return most >= 64 ? 4 : most >= 16 ? 2 : 1;
}

FusedPlan plan_fused(const chunk_attn_desc* d, int keys, int num_xcd, int num_bufs) {
  FusedPlan P;
  P.num_bufs = num_bufs;
  struct Chain { int first_item, n_items; int64_t work; };
  std::vector<Chain> chains;
  int32_t q_tile0 = 0, dq_tile0 = 0;
  for (int t = 0; t < d->num_segments; ++t) {
    const chunk_attn_seg& s = d->segments[t];
    const int32_t C = s.kv_len - s.q_len;
    const int32_t n_qt = (s.q_len + 31) / 32;
    for (int kvh = 0; kvh < d->num_kv_heads; ++kvh) {
      Chain ch{(int)P.items.size(), 0, 0};
      int32_t b = 0;
      for (int32_t j0 = 0; j0 < s.kv_len; j0 += keys, ++b) {
        FusedItem it{};
        it.kv_row0 = s.kv_start + j0;
        it.kv_rows = std::min<int32_t>(keys, s.kv_len - j0);
        it.j0 = j0;
        it.ctx = C;
        it.q_row_seg = s.q_start;
        it.q_len = s.q_len;
        it.qt_first = std::max<int32_t>(0, j0 - C) / 32;
        it.n_qt = n_qt;
        it.q_tile0 = q_tile0;
        it.kvh = kvh;
        it.buf = b % num_bufs;
        it.pred = b < num_bufs ? -1 : (int32_t)P.items.size() - num_bufs;   // the block num_bufs before it: same sub-chain
        it.delta_qt = b < num_bufs ? 0 : it.qt_first - P.items[it.pred].qt_first;
        it.dq_tile0 = dq_tile0;
        ch.work += n_qt - it.qt_first;
        ++ch.n_items;
        P.items.push_back(it);
      }
      chains.push_back(ch);
    }
    for (int32_t qt = 0; qt < n_qt; ++qt)
      P.tiles.push_back(DqTileJob{s.q_start + 32 * qt, std::min<int32_t>(32, s.q_len - 32 * qt), dq_tile0 + qt, qt, C,
                                  (s.kv_len + keys - 1) / keys, 0, 0});
    q_tile0 += (s.q_len + 63) / 64;
    dq_tile0 += n_qt;
  }
  P.total_qt32 = dq_tile0;
  // chains to XCDs: most work first, each to the XCD with the least work so far
  std::vector<int> by_work(chains.size());
  for (size_t i = 0; i < chains.size(); ++i) by_work[i] = (int)i;
  std::stable_sort(by_work.begin(), by_work.end(), [&](int a, int b) { return chains[a].work > chains[b].work; });
  std::vector<int64_t> load(num_xcd, 0);
  std::vector<std::vector<int32_t>> lists(num_xcd);
  for (int c : by_work) {
    int x = 0;
    for (int i = 1; i < num_xcd; ++i)
      if (load[i] < load[x]) x = i;
    load[x] += chains[c].work;
    for (int i = 0; i < chains[c].n_items; ++i) lists[x].push_back(chains[c].first_item + i);
  }
  // inside an XCD: longest walk first; the walks of a chain do not grow along it, and the sort is stable, so a block
  // always comes after its predecessor
  size_t longest = 0;
  for (auto& l : lists) {
    std::stable_sort(l.begin(), l.end(), [&](int32_t a, int32_t b) {
      return P.items[a].n_qt - P.items[a].qt_first > P.items[b].n_qt - P.items[b].qt_first;
    });
    longest = std::max(longest, l.size());
  }
  P.order.assign(longest * num_xcd, -1);
  for (int x = 0; x < num_xcd; ++x)
    for (size_t i = 0; i < lists[x].size(); ++i) P.order[i * num_xcd + x] = lists[x][i];
  return P;
}

std::vector<std::pair<int32_t, int32_t>> uncovered_kv_ranges(const chunk_attn_desc* d) {
  std::vector<std::pair<int32_t, int32_t>> gaps;
  int32_t next = 0;
  for (int t = 0; t < d->num_segments; ++t) {
    const chunk_attn_seg& s = d->segments[t];
    if (s.kv_start > next) gaps.push_back({next, s.kv_start});
    next = s.kv_start + s.kv_len;
  }
  if (next < d->total_kv) gaps.push_back({next, d->total_kv});
  return gaps;
}

}  // namespace chunk_attn
