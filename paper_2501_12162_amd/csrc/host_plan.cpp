// Host-only part of the library (see host_plan.h): argument validation and
// the split-KV planner of the tree-attention entry points.
#include "host_plan.h"

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <iterator>
#include <string>

namespace adaserve {

namespace {
thread_local std::string g_last_error;
}  // namespace

int32_t fail(int32_t code, const char *fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  g_last_error = buf;
  return code;
}

const char *last_error_message() { return g_last_error.c_str(); }

size_t round_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Scalar and host-mirror validation shared by the workspace query and the
// verify call.  Does not touch device memory.
int32_t validate_attn_shape(int32_t num_requests, const int32_t *indptr_host, const int32_t *plen_host,
                            int32_t hq, int32_t hkv, int32_t head_dim, int32_t page_size, int32_t dtype,
                            int32_t bt_stride_or_neg, AttnShape &shape) {
  if (num_requests < 0) return fail(ADASERVE_ERR_INVALID_ARGUMENT, "num_requests %d < 0", num_requests);
  if (hq <= 0 || hkv <= 0) return fail(ADASERVE_ERR_INVALID_ARGUMENT, "head counts must be positive (%d, %d)", hq, hkv);
  if (hq % hkv != 0)
    return fail(ADASERVE_ERR_INVALID_ARGUMENT, "num_q_heads %d is not a multiple of num_kv_heads %d", hq, hkv);
  if (hq / hkv > 16) return fail(ADASERVE_ERR_UNSUPPORTED, "head group %d > 16", hq / hkv);
  if (dtype != ADASERVE_F32 && dtype != ADASERVE_BF16) return fail(ADASERVE_ERR_INVALID_ARGUMENT, "unknown dtype %d", dtype);
  if (head_dim != 64 && head_dim != 128) return fail(ADASERVE_ERR_UNSUPPORTED, "head_dim %d (supported: 64, 128)", head_dim);
  if (page_size != kPageSize) return fail(ADASERVE_ERR_UNSUPPORTED, "page_size %d (supported: 16)", page_size);
  shape.num_requests = num_requests;
  shape.group = hq / hkv;
  if (num_requests == 0) return ADASERVE_OK;
  if (!indptr_host || !plen_host) return fail(ADASERVE_ERR_INVALID_ARGUMENT, "host mirrors must not be NULL");
  if (indptr_host[0] != 0) return fail(ADASERVE_ERR_INVALID_ARGUMENT, "node_indptr[0] = %d, expected 0", indptr_host[0]);
  int64_t total = 0;
  for (int32_t r = 0; r < num_requests; ++r) {
    const int64_t n = (int64_t)indptr_host[r + 1] - indptr_host[r];
    if (n < 1) return fail(ADASERVE_ERR_INVALID_ARGUMENT, "request %d has %lld tree nodes (need >= 1)", r, (long long)n);
    if (n > kMaxTreeNodes) return fail(ADASERVE_ERR_UNSUPPORTED, "request %d has %lld tree nodes (max %d)", r, (long long)n, kMaxTreeNodes);
    total += n;
    const int32_t L = plen_host[r];
    if (L < 0) return fail(ADASERVE_ERR_INVALID_ARGUMENT, "prefix_len[%d] = %d < 0", r, L);
    if (L > kMaxPrefixLen) return fail(ADASERVE_ERR_UNSUPPORTED, "prefix_len[%d] = %d (max %d)", r, L, kMaxPrefixLen);
    if (bt_stride_or_neg >= 0 && ceil_div(L, kPageSize) > bt_stride_or_neg)
      return fail(ADASERVE_ERR_INVALID_ARGUMENT, "prefix_len[%d] = %d needs %d pages > block_table_stride %d", r, L,
                  ceil_div(L, kPageSize), bt_stride_or_neg);
  }
  if (total > INT32_MAX / 16) return fail(ADASERVE_ERR_INVALID_ARGUMENT, "too many tree nodes (%lld)", (long long)total);
  shape.total_nodes = (int32_t)total;
  return ADASERVE_OK;
}

// Cost model of the bf16 kernel on MI355X.
//  * A call costs kCallUs around its steps (launch, start-up loads, output
//    writes) and kCombineUs when a prefix is split (the merge).
//  * Up to two units per CU (one round): a CU streams kCuBytesPerUs with one
//    unit and is credited kPairBytesPerUs more with two (above the measured
//    2-3e3: more streams also even out slow XCDs); a 32-key step of a unit
//    alone on its CU takes kStepUs, a step of a second unit beside it kPairUs
//    and kPairWaveUs for each of its live waves (32 rows).
//    Units past the first kFreeStarts hold up each other's first blocks by
//    kUnitStartUs each.  Short launches run at a higher clock (2.7 GHz against
//    2.1-2.2 from ~100 us on), which prices the second unit's share down to
//    kShortClock.
//  * More units (several rounds): kUnitFixedUs per unit and kBlockUs per step,
//    dealt longest first, and kChipBytesPerUs.  Head_dim 64 is always priced
//    this way, streaming by the share of the slots that the units fill.
// Only kStepUs, kChipBytesPerUs, kCombineUs and the clocks were measured by
// themselves; kPairBytesPerUs, kFreeStarts, kUnitStartUs, kPairUs, kPairWaveUs
// and kTileReread are set so that the estimates order such sweeps (estimate |
// measured, us): attention of the 16-request 8B batch in 200 units 49.1 | 45.5,
// 328 38.6 | 39.0, 512 35.6 | 39.2; a rank of the 70B shape in 294 212 | 167,
// 512 129 | 115-117; long context in 256 203 | 209, 448 178 | 197, 512 159 |
// 195.  They rank the splits of one batch and are not times.  Least so at
// head_dim 64, where the model has two resident units per CU of 1 us a step
// and the present kernel (124 VGPRs, 40 KB of LDS) four: 25 requests of 62587
// keys in 1056 units 767 | 349, in 4092 586 | 334.
constexpr double kCallUs = 6.0;
constexpr double kUnitStartUs = 0.02;
constexpr int kFreeStarts = 167;
constexpr double kCombineUs = 3.0;
constexpr double kCuBytesPerUs = 22.0e3;
constexpr double kPairBytesPerUs = 7.2e3;
constexpr double kCuMostBytesPerUs = 30.0e3;   // of one CU while others are done
constexpr double kBytesPerStep = 32 * 512.0;    // K and V at head_dim 128
constexpr double kTileReread = 0.3;   // HBM cost of a chunk's further row tiles (most hit L2)
constexpr double kStepUs = 0.72;
constexpr double kPairUs = 0.1;
constexpr double kPairWaveUs = 0.03;
constexpr double kShortClock = 0.78;
constexpr double kChipBytesPerUs = 5.8e6;
constexpr double kBlockUs = 1.0;
constexpr double kUnitFixedUs = 6.0;
constexpr int kCUs = 256;
constexpr int kSlots = 2 * kCUs;  // resident workgroups: two per CU

// Makespan of units dispatched longest first onto kSlots workgroup slots,
// each unit taking the slot that frees up first (how the hardware deals a
// grid whose units come in that order).  Slot loads are kept as runs of
// equal load, so the cost grows with the number of distinct durations, not
// with the number of units.  `units` holds (duration, count) pairs in any
// order; it is sorted in place.
using Durations = std::vector<std::pair<double, int64_t>>;
static double deal_longest_first(const Durations &units, Durations &runs, double limit);

double lpt_makespan(Durations &units) {
  std::sort(units.begin(), units.end(), [](const auto &x, const auto &y) { return x.first > y.first; });
  size_t m = 0;  // merge equal durations
  for (size_t i = 0; i < units.size(); ++i) {
    if (m > 0 && units[m - 1].first == units[i].first)
      units[m - 1].second += units[i].second;
    else
      units[m++] = units[i];
  }
  units.resize(m);
  Durations runs;
  return deal_longest_first(units, runs, HUGE_VAL);
}

// The same for distinct durations in descending order; a makespan past `limit`
// may be returned short, but still past it.  `runs` is scratch.
static double deal_longest_first(const Durations &units, Durations &runs, double limit) {
  runs.clear();
  runs.push_back({0.0, (int64_t)kSlots});  // (load, slots), ascending from runs[head]
  size_t head = 0;
  auto insert = [&](double load, int64_t slots) {
    // most new loads are among the highest
    size_t i = runs.size();
    while (i > head && runs[i - 1].first > load) --i;
    if (i > head && runs[i - 1].first == load)
      runs[i - 1].second += slots;
    else
      runs.insert(runs.begin() + i, {load, slots});
  };
  for (const auto &u : units) {
    const double t = u.first;
    int64_t c = u.second;
    // Units of duration t go one by one to a least-loaded slot.  The k0
    // slots of the lowest run take them in rounds, one per slot, until they
    // pass the next run's load (or the units run out): whole rounds move the
    // run up together; a last partial round splits it.
    while (c > 0) {
      const double x0 = runs[head].first;
      const int64_t k0 = runs[head].second;
      if (c < k0) {
        runs[head].second -= c;
        insert(x0 + t, c);
        break;
      }
      ++head;
      int64_t rounds = 1;
      if (c >= 2 * k0) {
        rounds = c / k0;
        if (head < runs.size())
          rounds = std::min<int64_t>(rounds, std::max<int64_t>(1, (int64_t)std::ceil((runs[head].first - x0) / t)));
      }
      c -= rounds * k0;
      insert(x0 + (double)rounds * t, k0);
    }
    if (runs.back().first > limit) break;
  }
  return runs.back().first;
}

// Buffers that the pricing of a batch's choices shares.
struct PricingScratch {
  std::vector<UnitRun> units;   // longest first
  std::vector<int32_t> steps, chunks;
  Durations timed, runs;
};

// The time of one CU's units: `first` alone, or with `second` beside it.
double pair_us(const UnitRun &first, const UnitRun *second) {
  const double own = first.steps * first.share, other = second ? second->steps * second->share : 0.0;
  const double alone = first.steps * kStepUs;
  const double clock = kShortClock + (1.0 - kShortClock) * std::min(1.0, alone / 60.0);
  return std::max((own + other) * kBytesPerStep / kCuMostBytesPerUs,
                  alone + (second ? second->steps * (kPairUs + second->live * kPairWaveUs) * clock : 0.0));
}

double one_round_us(const std::vector<UnitRun> &units, int64_t total) {
  double worst = 0;
  // walk unit i and its partner kCUs + i through the runs together
  size_t p = 0;
  int64_t p_left = 0, skip = kCUs;
  for (; p < units.size(); ++p) {
    if (skip < units[p].count) {
      p_left = units[p].count - skip;
      break;
    }
    skip -= units[p].count;
  }
  int64_t placed = 0;
  for (size_t i = 0; i < units.size() && placed < kCUs; ++i) {
    int64_t left = std::min<int64_t>(units[i].count, kCUs - placed);
    placed += left;
    while (left > 0) {
      const bool pair = p < units.size();
      const int64_t take = pair ? std::min(left, p_left) : left;
      worst = std::max(worst, pair_us(units[i], pair ? &units[p] : nullptr));
      left -= take;
      if (pair && (p_left -= take) == 0 && ++p < units.size()) p_left = units[p].count;
    }
  }
  return worst + kUnitStartUs * std::max<int64_t>(0, total - kFreeStarts);
}

// Time the steps of `w.units` take: one round (at most kSlots units) by
// one_round_us, several rounds by longest-first dealing (a time past `limit`
// may be returned short, but still past it).
static double steps_us(PricingScratch &w, int64_t total, int32_t head_dim, double limit) {
  if (total <= kSlots && head_dim != 64) return one_round_us(w.units, total);
  w.timed.clear();
  for (const UnitRun &u : w.units) {
    const double t = kUnitFixedUs + u.steps * kBlockUs;
    if (!w.timed.empty() && w.timed.back().first == t)
      w.timed.back().second += u.count;
    else
      w.timed.push_back({t, u.count});
  }
  return deal_longest_first(w.timed, w.runs, limit);
}

// Workspace of a plan that splits a prefix: per unit, kMaxRowsPerTile bf16 output
// rows, then fp32 (max, denominator) pairs.
static size_t partial_rows_bytes(int64_t units, int32_t head_dim) {
  return round_up((size_t)units * kMaxRowsPerTile * head_dim * 2, 256);
}
static size_t partial_bytes(int64_t units, int32_t head_dim) {
  return partial_rows_bytes(units, head_dim) + round_up((size_t)units * kMaxRowsPerTile * 2 * sizeof(float), 256);
}

// ceil(a / b) by a float division, several times as fast as an integer one:
// exact while a + b < 2^22 (block counts are at most 2^18), where the quotient
// stays at least 0.5 / b off the integers and rounds by less.
static inline int32_t quick_ceil_div(int32_t a, int32_t b) {
  return (int32_t)(((float)(a + b) - 0.5f) / (float)b);
}

// Blocks of the tree in a chunk's steps: the at most 4 tree blocks are spread
// over the chunks.
static inline int32_t tree_steps(int32_t tree_blocks, int32_t chunks) {
  return 1 + (tree_blocks > chunks) + (tree_blocks > 2 * chunks) + (tree_blocks > 3 * chunks);
}

// What the plan choices of a batch share: the sizes of each request, in the
// bf16 kernel's units.
struct PlanRequest {
  int32_t blocks, tree_blocks;   // of 32 keys: prefix and tree
  int32_t tiles, full;           // row tiles, and how many of them are full
  int32_t last_live;             // live waves of the last, partial one (0: none)
  int32_t floor_rows;            // rows of a tile, for chunk_keys()
  double share;                  // of a chunk's K/V bytes that one tile streams from HBM
  int64_t head_tiles;            // kv-heads * row tiles
  double chunk_partials;         // bytes of split-KV partials of one chunk
};

// `kv_bytes`: what the batch's units stream of K and V, however it is split.
static std::vector<PlanRequest> plan_requests(int32_t B, const int32_t *indptr_host, const int32_t *plen_host,
                                              int32_t hkv, int32_t group, int32_t head_dim, double &kv_bytes) {
  constexpr int32_t rt = kMaxRowsPerTile;
  const double key_bytes = 4.0 * head_dim;  // bf16 K and V of one key of one kv-head
  std::vector<PlanRequest> reqs(B);
  kv_bytes = 0;
  for (int32_t r = 0; r < B; ++r) {
    PlanRequest &q = reqs[r];
    const int32_t n = indptr_host[r + 1] - indptr_host[r];
    const int32_t rows = n * group;
    q.blocks = ceil_div(plen_host[r], kKeysPerBlock);
    q.tree_blocks = ceil_div(n, kKeysPerBlock);
    q.tiles = row_tiles(n, group, rt);
    q.full = rows / rt;
    q.last_live = ceil_div(rows % rt, 32);
    q.floor_rows = std::min(rows, rt);
    const double streamed = 1.0 + kTileReread * (q.tiles - 1);
    q.share = streamed / q.tiles;
    q.head_tiles = (int64_t)hkv * q.tiles;
    q.chunk_partials = hkv * (double)rows * (head_dim * 2.0 + 8.0);
    kv_bytes += (double)hkv * streamed * (plen_host[r] + n) * key_bytes;
  }
  return reqs;
}

// One choice of chunk lengths and what it costs apart from its steps.
struct PlanChoice {
  size_t ck;            // its chunk lengths, as an offset
  int32_t fm, c;        // batch-wide family (fm = 0: balanced)
  int64_t units;
  bool split;
  double stream, fixed; // streaming time (K/V plus the split partials); kCallUs and the merge
  double bound;         // a lower bound of the estimate
};

// Prices the choice of chunk lengths `ck` (prefix keys per unit, whole 32-key
// blocks, at most kMaxChunk) with 128-row tiles.  The estimate is `fixed` plus
// the larger of `stream` and the steps' time (steps_us); `bound` puts a lower
// bound in the place of the latter: in one round the longest unit beside the
// shortest, in several the longest unit, the rounds of the shortest, or the
// mean load of the slots.
static PlanChoice price_choice(const std::vector<PlanRequest> &reqs, const int32_t *ck, int32_t head_dim,
                               double kv_bytes) {
  PlanChoice p{};
  double partial_bytes = 0;
  int32_t longest = 0, shortest = INT32_MAX;
  int64_t steps_total = 0;
  for (size_t r = 0; r < reqs.size(); ++r) {
    const PlanRequest &q = reqs[r];
    const int32_t per_chunk = ck[r] / kKeysPerBlock;
    int32_t steps;
    if (q.blocks <= per_chunk) {
      steps = q.blocks + q.tree_blocks;
      p.units += q.head_tiles;
      steps_total += q.head_tiles * steps;
    } else {
      const int32_t chunks = quick_ceil_div(q.blocks, per_chunk);
      steps = per_chunk + tree_steps(q.tree_blocks, chunks);
      p.split = true;
      partial_bytes += chunks * q.chunk_partials;
      p.units += q.head_tiles * chunks;
      steps_total += q.head_tiles * chunks * steps;
    }
    longest = std::max(longest, steps);
    shortest = std::min(shortest, steps);
  }
  const double alone = (double)std::min<int64_t>(p.units, kCUs);
  const double paired = (double)std::min<int64_t>(std::max<int64_t>(p.units - kCUs, 0), kCUs);
  const bool one_round = head_dim != 64 && p.units <= kSlots;
  const double rate = one_round ? alone * kCuBytesPerUs + paired * kPairBytesPerUs
                                : kChipBytesPerUs * (alone + paired) / kSlots;
  p.fixed = kCallUs + (p.split ? kCombineUs + partial_bytes / rate : 0.0);
  p.stream = (kv_bytes + partial_bytes) / rate;
  double steps_bound;
  if (one_round) {
    steps_bound = longest * kStepUs + (p.units > kCUs ? shortest * (kPairUs + kPairWaveUs) * kShortClock : 0.0) +
                  kUnitStartUs * std::max<int64_t>(0, p.units - kFreeStarts);
  } else {
    const int64_t rounds = (p.units + kSlots - 1) / kSlots;   // units of the busiest slot, at least
    steps_bound = std::max({kUnitFixedUs + longest * kBlockUs, rounds * (kUnitFixedUs + shortest * kBlockUs),
                            (kUnitFixedUs * (double)p.units + (double)steps_total * kBlockUs) / kSlots});
  }
  p.bound = std::max(p.stream, steps_bound) + p.fixed;
  return p;
}

// The units of a choice in descending order of steps (requests of equal steps
// in their order), for steps_us.
static void list_units(const std::vector<PlanRequest> &reqs, const int32_t *ck, int32_t hkv, PricingScratch &w) {
  constexpr int32_t kMost = (kMaxChunk + kMaxTreeNodes) / kKeysPerBlock;   // steps of a unit
  int32_t at[kMost + 2] = {};
  const size_t B = reqs.size();
  w.steps.resize(B);
  w.chunks.resize(B);
  for (size_t r = 0; r < B; ++r) {
    const PlanRequest &q = reqs[r];
    const int32_t per_chunk = ck[r] / kKeysPerBlock;
    const int32_t chunks = q.blocks <= per_chunk ? 1 : quick_ceil_div(q.blocks, per_chunk);
    const int32_t steps = std::min(q.blocks, per_chunk) + tree_steps(q.tree_blocks, chunks);
    w.chunks[r] = chunks;
    w.steps[r] = steps;
    at[kMost - steps + 1] += (q.full > 0) + (q.last_live > 0);
  }
  for (int32_t i = 0; i <= kMost; ++i) at[i + 1] += at[i];
  w.units.resize(at[kMost + 1]);
  for (size_t r = 0; r < B; ++r) {
    const PlanRequest &q = reqs[r];
    const int64_t each = (int64_t)hkv * w.chunks[r];
    int32_t &i = at[kMost - w.steps[r]];
    if (q.full > 0) w.units[i++] = {w.steps[r], kMaxRowsPerTile / 32, q.share, each * q.full};
    if (q.last_live > 0) w.units[i++] = {w.steps[r], q.last_live, q.share, each};
  }
}

double estimate_plan(int32_t B, const int32_t *indptr_host, const int32_t *plen_host, int32_t hkv, int32_t group,
                     int32_t head_dim, const int32_t *chunk_len) {
  double kv_bytes;
  const std::vector<PlanRequest> reqs = plan_requests(B, indptr_host, plen_host, hkv, group, head_dim, kv_bytes);
  const PlanChoice c = price_choice(reqs, chunk_len, head_dim, kv_bytes);
  PricingScratch w;
  list_units(reqs, chunk_len, hkv, w);
  return std::max(c.stream, steps_us(w, c.units, head_dim, HUGE_VAL)) + c.fixed;
}

// Work plan of the F32 kernel: 32-row tiles when they alone give every CU a
// unit, else 16-row tiles (twice the units, each K/V byte read twice as
// often).  Requests of 8-64 nodes over 64-1024 keys, 16 / 4 heads, D = 128,
// 16- against 32-row tiles: 72 units of 32 rows 30.7 / 50.0 us, 228 46.8 /
// 51.0, 328 64.7 / 58.4, 956 154 / 138.
static AttnPlan make_f32_plan(int32_t B, const int32_t *indptr_host, int32_t hkv, int32_t group) {
  AttnPlan p;
  auto count = [&](int32_t rt) {
    int64_t units = 0;
    for (int32_t r = 0; r < B; ++r) units += (int64_t)hkv * row_tiles(indptr_host[r + 1] - indptr_host[r], group, rt);
    return units;
  };
  p.rows_per_tile = count(32) >= kCUs ? 32 : 16;
  p.units = p.row_groups = count(p.rows_per_tile);
  p.padded_grid = pad_to_xcds(p.units);
  p.chunk_target = kF32Chunk;
  p.chunk_floor = 1;
  p.chunk_len.assign(B, kF32Chunk);
  return p;
}

// Work plan of the bf16 kernel, from host-visible sizes only: the cheapest
// estimate over two families of prefix splits, 128-row tiles.  (A 64-row
// tile costs about as much per step as a 128-row one, so it never wins.)
//  * batch-wide chunk targets {256 .. 8192} with chunk floors {8, 16, 32}
//    keys per row (chunk_keys() in plan.h), the only family the device can
//    rebuild without a plan table;
//  * with a plan table, balanced splits: for a target unit count, every
//    request's prefix is cut into the fewest equal runs of whole 32-key
//    blocks no longer than the batch's mean blocks per unit, so the units
//    come out about equally long and fill the workgroup slots evenly.
// Choices that give every request the same chunk lengths as one already
// tried, or split nothing as one did, are skipped, and the steps are only timed for choices whose lower
// bound can still be taken.  Requests are then dispatched in descending order
// of per-unit cost (fill_plan_table).
AttnPlan make_plan(int32_t B, const int32_t *indptr_host, const int32_t *plen_host, int32_t hkv,
                   int32_t group, int32_t head_dim, int32_t dtype, bool in_scratch) {
  AttnPlan best;
  if (B == 0) return best;
  if (dtype != ADASERVE_BF16) return make_f32_plan(B, indptr_host, hkv, group);
  constexpr int32_t rt = kMaxRowsPerTile;
  constexpr int32_t kFloors[] = {32, 16, 8};
  constexpr int32_t kTargets[] = {160, 192, 224, 256, 288, 320, 352, 384, 416, 448, 512, 576, 640, 768, 1024};
  double kv_bytes;
  const std::vector<PlanRequest> reqs = plan_requests(B, indptr_host, plen_host, hkv, group, head_dim, kv_bytes);
  int64_t work = 0;   // unit-blocks of the unsplit batch
  for (const PlanRequest &q : reqs) work += q.head_tiles * std::max(1, q.blocks);

  std::vector<PlanChoice> choices;
  choices.reserve(std::size(kFloors) * 6 + std::size(kTargets));
  std::vector<int32_t> cks;   // chunk lengths of all choices, and of the one being made
  cks.reserve((choices.capacity() + 1) * B);
  auto add = [&](int32_t fm, int32_t c) {
    const int32_t *ck = cks.data() + cks.size() - B;
    PlanChoice p = price_choice(reqs, ck, head_dim, kv_bytes);
    for (const PlanChoice &x : choices)
      if (x.units == p.units && x.bound == p.bound &&
          ((!x.split && !p.split) || std::equal(ck, ck + B, cks.data() + x.ck))) {
        cks.resize(cks.size() - B);
        return;
      }
    p.ck = cks.size() - B;
    p.fm = fm;
    p.c = c;
    choices.push_back(p);
  };
  int32_t longest_prefix = 0;
  for (const PlanRequest &q : reqs) longest_prefix = std::max(longest_prefix, q.blocks * kKeysPerBlock);
  bool unsplit = false;   // one choice that splits nothing is enough
  auto splits_nothing_again = [&](int32_t chunk) { return chunk >= longest_prefix && std::exchange(unsplit, true); };
  std::vector<int32_t> floor_ck(B);
  int32_t above = INT32_MAX;   // from this target on the floors have no effect: the same as with the last floor
  for (int32_t fm : kFloors) {
    int32_t least_floor = INT32_MAX, most_floor = 0;
    for (int32_t r = 0; r < B; ++r) {
      floor_ck[r] = chunk_keys(1, reqs[r].floor_rows, rt, 0, fm);
      least_floor = std::min(least_floor, floor_ck[r]);
      most_floor = std::max(most_floor, floor_ck[r]);
    }
    for (int32_t c = kMaxChunk; c >= kMinChunk; c /= 2) {
      if (c >= above || 2 * c <= least_floor || splits_nothing_again(c)) continue;
      for (int32_t r = 0; r < B; ++r) cks.push_back(std::max(floor_ck[r], c));
      add(fm, c);
    }
    above = most_floor;
  }
  if (B <= kPlanMax) {
    int32_t last = 0;
    for (int32_t target : kTargets) {
      const int32_t per_unit =
          (int32_t)std::min<int64_t>(std::max<int64_t>(4, (work + target - 1) / target), kMaxChunk / kKeysPerBlock);
      if (per_unit == last || splits_nothing_again(per_unit * kKeysPerBlock)) continue;
      last = per_unit;
      for (const PlanRequest &q : reqs)
        cks.push_back(q.blocks == 0 ? kMaxChunk
                                    : quick_ceil_div(q.blocks, quick_ceil_div(q.blocks, per_unit)) * kKeysPerBlock);
      add(0, 0);
    }
  }
  std::vector<std::pair<double, size_t>> order;   // (bound, choice), ascending
  order.reserve(choices.size());
  for (size_t i = 0; i < choices.size(); ++i) order.push_back({choices[i].bound, i});
  std::sort(order.begin(), order.end());

  // The cheapest estimate wins; at head_dim 128, among plans of more than a
  // unit per CU within kTie of it (what the estimate is good for), the one of
  // fewest units: it has less to merge, and in the one-call step the argmax
  // rows find free slots from the start.  (Step of the 8B batch: 512 units
  // 66.2 us, 464 64.2, 440 59.5, 416 58-59; its attention alone 36-39 for all.)
  constexpr double kTie = 1.1;
  PricingScratch w;
  std::vector<double> ests(choices.size(), 0.0);   // 0: not priced yet
  // The estimate of choice i, or something past `limit` when it is past that.
  auto estimate = [&](size_t i, double limit) {
    if (ests[i] == 0.0) {
      const PlanChoice &c = choices[i];
      list_units(reqs, cks.data() + c.ck, hkv, w);
      const double est = std::max(c.stream, steps_us(w, c.units, head_dim, limit - c.fixed)) + c.fixed;
      if (est > limit) return est;
      ests[i] = est;
    }
    return ests[i];
  };
  auto fits = [&](const PlanChoice &c) {
    return !c.split || partial_bytes(c.units, head_dim) <= ADASERVE_TREE_ATTN_SCRATCH_BYTES;
  };
  constexpr size_t kNone = SIZE_MAX;
  // The choice taken (of those whose partials fit the static scratch, with
  // `fit_only`; kNone when none does), and the one of the least estimate.
  auto select = [&](bool fit_only, size_t &cheapest) {
    size_t pick = kNone;
    for (const auto &[bound, i] : order) {
      if (pick != kNone && bound >= ests[pick]) break;   // none of the rest is cheaper
      if (fit_only && !fits(choices[i])) continue;
      const double most = pick == kNone ? HUGE_VAL : ests[pick];
      if (estimate(i, most) < most) pick = i;
    }
    cheapest = pick;
    if (pick == kNone) return pick;
    if (head_dim != 128 || choices[pick].units <= kCUs) return pick;
    const double tie = ests[pick] * kTie;
    std::vector<std::pair<int64_t, size_t>> fewer;   // (units, choice), ascending
    for (const auto &[bound, i] : order)
      if (bound <= tie && choices[i].units > kCUs && choices[i].units < choices[pick].units &&
          (!fit_only || fits(choices[i])))
        fewer.push_back({choices[i].units, i});
    std::sort(fewer.begin(), fewer.end());
    size_t fewest = kNone;
    for (const auto &[few, i] : fewer) {
      if (fewest != kNone && few > choices[fewest].units) break;
      const double most = fewest == kNone ? tie : ests[fewest];
      if (estimate(i, most) <= most && (fewest == kNone || ests[i] < ests[fewest])) fewest = i;
    }
    return fewest == kNone ? pick : fewest;
  };
  size_t cheapest = kNone;
  size_t pick = select(false, cheapest);
  // Plans whose partials fit the static scratch are taken as long as the least
  // estimate of them ties with the least of all, and by a call that has only
  // the scratch at up to kScratchCost times that.  (At a tie the estimates do
  // not tell which is faster, measured 0.91-1.11 either way; at 1.27 times,
  // 65 requests of 1-8 nodes over 6600 keys, 64 / 8 heads, 350 | 325 us with a
  // workspace.)
  constexpr double kScratchCost = 1.6;
  if (!fits(choices[cheapest])) {   // if it fits, so does a tie of fewer units
    size_t cheapest_fit = kNone;
    const size_t fit = select(true, cheapest_fit);
    if (fit != kNone && ests[cheapest_fit] <= ests[cheapest] * (in_scratch ? kScratchCost : kTie)) pick = fit;
  }
  const PlanChoice &chosen = choices[pick];
  best.rows_per_tile = rt;
  best.chunk_len.assign(cks.begin() + chosen.ck, cks.begin() + chosen.ck + B);
  best.units = chosen.units;
  best.padded_grid = pad_to_xcds(best.units);
  best.needs_combine = chosen.split;
  if (best.needs_combine) {
    best.ws_o_bytes = partial_rows_bytes(best.units, head_dim);
    best.ws_bytes = partial_bytes(best.units, head_dim);
    best.ws_ml_bytes = best.ws_bytes - best.ws_o_bytes;
  }
  best.est_us = ests[pick];
  // the batch-wide fields rebuild the chunks when there is no plan table
  best.chunk_target = chosen.fm ? chosen.c : kMaxChunk;
  best.chunk_floor = chosen.fm ? chosen.fm : 32;
  best.single_tile = true;
  for (const PlanRequest &q : reqs) {
    best.row_groups += q.head_tiles;
    best.single_tile &= q.tiles == 1;
  }
  return best;
}

AttnPlan make_plan_cached(int32_t B, const int32_t *indptr_host, const int32_t *plen_host, int32_t hkv,
                          int32_t group, int32_t head_dim, int32_t dtype, bool in_scratch) {
  if (dtype != ADASERVE_BF16 || B <= 0) return make_plan(B, indptr_host, plen_host, hkv, group, head_dim, dtype);
  struct Entry {
    bool valid = false;
    int32_t B = 0, hkv = 0, group = 0, head_dim = 0, dtype = 0;
    std::vector<int32_t> indptr, plen;
    AttnPlan plan;
  };
  thread_local Entry entries[2];
  Entry &e = entries[in_scratch];
  const bool hit = e.valid && e.B == B && e.hkv == hkv && e.group == group && e.head_dim == head_dim &&
                   e.dtype == dtype && std::equal(indptr_host, indptr_host + B + 1, e.indptr.begin()) &&
                   std::equal(plen_host, plen_host + B, e.plen.begin());
  if (!hit) {
    e.valid = false;
    e.plan = make_plan(B, indptr_host, plen_host, hkv, group, head_dim, dtype, in_scratch);
    e.indptr.assign(indptr_host, indptr_host + B + 1);
    e.plen.assign(plen_host, plen_host + B);
    e.B = B;
    e.hkv = hkv;
    e.group = group;
    e.head_dim = head_dim;
    e.dtype = dtype;
    e.valid = true;
  }
  return e.plan;
}

// Fills the dispatch-ordered request table (descending per-unit cost) when
// the batch fits in the kernel arguments; otherwise leaves it empty.
void fill_plan_table(PlanTable &t, int32_t B, const int32_t *indptr_host, const int32_t *plen_host,
                     int32_t num_kv_heads, int32_t group, const AttnPlan &p) {
  t.count = 0;
  t.merge_blocks = 0;
  if (B > kPlanMax) return;
  int32_t order[kPlanMax];
  int64_t cost[kPlanMax];
  for (int32_t r = 0; r < B; ++r) {
    const int32_t n = indptr_host[r + 1] - indptr_host[r];
    const int32_t keys = std::min(std::max(plen_host[r], 0), p.chunk_len[r]);
    cost[r] = keys + n;  // steps per unit (the step time hardly depends on the row count)
    order[r] = r;
  }
  std::stable_sort(order, order + B, [&](int32_t x, int32_t y) { return cost[x] > cost[y]; });
  int64_t end = 0, gend = 0;
  for (int32_t i = 0; i < B; ++i) {
    const int32_t r = order[i];
    const int32_t n = indptr_host[r + 1] - indptr_host[r];
    end += (int64_t)num_kv_heads * row_tiles(n, group, p.rows_per_tile) *
           prefix_chunks(plen_host[r], p.chunk_len[r]);
    // merge blocks: 16 rows of one kv-head each, for split requests only
    if (prefix_chunks(plen_host[r], p.chunk_len[r]) > 1) gend += (int64_t)num_kv_heads * ceil_div(n * group, 16);
    t.entry[i].unit_end = (int32_t)end;
    t.entry[i].group_end = (int32_t)gend;
    t.entry[i].request_and_chunk = pack_request_chunk(r, p.chunk_len[r]);
    t.entry[i].node_base = indptr_host[r];
    t.entry[i].n_and_len = pack_nodes_len(n, plen_host[r]);
  }
  t.count = B;
  t.merge_blocks = gend;
}


}  // namespace adaserve
