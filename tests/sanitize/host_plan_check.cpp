// Checks of the library's host-only code (argument validation, split-KV
// planner, plan-table packing), built with -fsanitize=address,undefined by
// tests/test_sanitizers.py.  Exits 1 on the first broken invariant; the
// sanitizers abort on any memory error or undefined behaviour.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <queue>
#include <random>
#include <set>
#include <vector>

#include "host_plan.h"

using namespace adaserve;

static int g_checks = 0;
#define CHECK(cond, ...)                                              \
  do {                                                                \
    ++g_checks;                                                       \
    if (!(cond)) {                                                    \
      std::fprintf(stderr, "FAILED %s:%d: %s: ", __FILE__, __LINE__, #cond); \
      std::fprintf(stderr, __VA_ARGS__);                              \
      std::fprintf(stderr, "\n");                                     \
      std::exit(1);                                                   \
    }                                                                 \
  } while (0)

struct Batch {
  std::vector<int32_t> indptr, plen;
};

static Batch random_batch(std::mt19937_64 &rng, int B, int max_nodes, int max_len) {
  Batch b;
  b.indptr.push_back(0);
  for (int r = 0; r < B; ++r) {
    const int n = 1 + (int)(rng() % (uint64_t)max_nodes);
    b.indptr.push_back(b.indptr.back() + n);
    int L;
    switch (rng() % 6) {
      case 0: L = 0; break;
      case 1: L = (int)(rng() % 64); break;
      case 2: L = 32 * (int)(rng() % 300) + (int)(rng() % 3) - 1; break;
      default: L = (int)(rng() % (uint64_t)(max_len + 1)); break;
    }
    b.plen.push_back(L < 0 ? 0 : L);
  }
  return b;
}

// Brute-force longest-first dealing onto kSlots equal slots (the planner's
// makespan model) with a heap.
static double brute_makespan(std::vector<std::pair<double, int64_t>> units, int slots) {
  std::vector<double> d;
  for (auto &u : units)
    for (int64_t i = 0; i < u.second; ++i) d.push_back(u.first);
  std::sort(d.begin(), d.end(), [](double x, double y) { return x > y; });
  std::priority_queue<double, std::vector<double>, std::greater<double>> q;
  for (int i = 0; i < slots; ++i) q.push(0.0);
  double mk = 0;
  for (double t : d) {
    double s = q.top();
    q.pop();
    s += t;
    mk = std::max(mk, s);
    q.push(s);
  }
  return mk;
}

static void check_plan(const Batch &b, int hq, int hkv, int D) {
  const int B = (int)b.plen.size();
  AttnShape shape;
  const int32_t st = validate_attn_shape(B, b.indptr.data(), b.plen.data(), hq, hkv, D, 16, ADASERVE_BF16, -1, shape);
  if (st != ADASERVE_OK) return;
  const int G = hq / hkv;
  const AttnPlan p = make_plan(B, b.indptr.data(), b.plen.data(), hkv, G, D, ADASERVE_BF16);
  CHECK((int)p.chunk_len.size() == B, "%zu chunk lengths for %d requests", p.chunk_len.size(), B);
  int64_t units = 0, groups = 0;
  bool split = false;
  for (int r = 0; r < B; ++r) {
    const int n = b.indptr[r + 1] - b.indptr[r];
    const int ck = p.chunk_len[r];
    CHECK(ck > 0 && ck <= kMaxChunk && ck % kKeysPerBlock == 0, "request %d chunk %d", r, ck);
    const int chunks = prefix_chunks(b.plen[r], ck);
    units += (int64_t)hkv * row_tiles(n, G, p.rows_per_tile) * chunks;
    groups += (int64_t)hkv * row_tiles(n, G, p.rows_per_tile);
    split |= chunks > 1;
    if (B > kPlanMax)  // without a plan table the device rebuilds the chunk lengths
      CHECK(ck == chunk_keys(n, G, p.rows_per_tile, p.chunk_target, p.chunk_floor), "request %d", r);
  }
  CHECK(units == p.units, "units %lld vs %lld", (long long)units, (long long)p.units);
  CHECK(groups == p.row_groups, "row groups");
  CHECK(split == p.needs_combine, "combine flag");
  bool one_tile = true;
  for (int r = 0; r < B; ++r) one_tile &= row_tiles(b.indptr[r + 1] - b.indptr[r], G, p.rows_per_tile) == 1;
  CHECK(one_tile == p.single_tile, "single-tile flag");
  CHECK((p.ws_bytes == 0) == !split, "workspace %zu", p.ws_bytes);
  if (split) {
    CHECK(p.ws_o_bytes >= (size_t)p.units * kMaxRowsPerTile * D * 2, "partial outputs");
    CHECK(p.ws_ml_bytes >= (size_t)p.units * kMaxRowsPerTile * 8, "partial max / sums");
    CHECK(p.ws_bytes == p.ws_o_bytes + p.ws_ml_bytes && p.ws_o_bytes % 256 == 0, "workspace layout");
  }
  CHECK(std::isfinite(p.est_us) && p.est_us > 0, "estimate %g", p.est_us);
  CHECK(p.padded_grid >= p.units && p.padded_grid % (kXcds * kXcdRun) == 0, "grid");
  if (p.padded_grid <= 4096) {
    std::vector<char> seen((size_t)p.padded_grid, 0);
    for (int64_t blk = 0; blk < p.padded_grid; ++blk) {
      const int64_t u = xcd_swizzle(blk, p.padded_grid);
      CHECK(u >= 0 && u < p.padded_grid && !seen[(size_t)u], "swizzle of %lld", (long long)blk);
      seen[(size_t)u] = 1;
    }
  }
  PlanTable t;
  fill_plan_table(t, B, b.indptr.data(), b.plen.data(), hkv, G, p);
  if (B > kPlanMax) {
    CHECK(t.count == 0, "table for %d requests", B);
    return;
  }
  CHECK(t.count == B, "table count");
  std::set<int> reqs;
  int64_t prev_end = 0, prev_g = 0, prev_cost = INT64_MAX;
  for (int i = 0; i < B; ++i) {
    const PlanEntry &e = t.entry[i];
    const int r = plan_request(e.request_and_chunk);
    CHECK(r >= 0 && r < B && reqs.insert(r).second, "entry %d request %d", i, r);
    const int n = b.indptr[r + 1] - b.indptr[r];
    CHECK(plan_nodes(e.n_and_len) == n, "nodes of %d", r);
    CHECK(plan_prefix_len(e.n_and_len) == b.plen[r], "prefix of %d", r);
    CHECK(plan_chunk_keys(e.request_and_chunk) == p.chunk_len[r], "chunk of %d", r);
    CHECK(e.node_base == b.indptr[r], "node base of %d", r);
    const int chunks = prefix_chunks(b.plen[r], p.chunk_len[r]);
    CHECK(e.unit_end - prev_end == (int64_t)hkv * row_tiles(n, G, p.rows_per_tile) * chunks, "units of %d", r);
    CHECK(e.group_end - prev_g == (chunks > 1 ? (int64_t)hkv * ceil_div(n * G, 16) : 0), "merge blocks of %d", r);
    const int64_t cost = std::min(b.plen[r], p.chunk_len[r]) + n;
    CHECK(cost <= prev_cost, "dispatch order at %d", i);
    prev_end = e.unit_end;
    prev_g = e.group_end;
    prev_cost = cost;
  }
  CHECK(prev_end == p.units && prev_g == t.merge_blocks, "table totals");
}

// F32 plans: whole prefixes, 32-row tiles where they give every CU a unit, no
// workspace, and a table that hands every field back.
static void check_f32_plan(const Batch &b, int hq, int hkv, int D) {
  const int B = (int)b.plen.size(), G = hq / hkv;
  AttnShape shape;
  if (validate_attn_shape(B, b.indptr.data(), b.plen.data(), hq, hkv, D, 16, ADASERVE_F32, -1, shape) != ADASERVE_OK)
    return;
  const AttnPlan p = make_plan(B, b.indptr.data(), b.plen.data(), hkv, G, D, ADASERVE_F32);
  int64_t units[2] = {0, 0};   // of 16 and of 32 rows
  for (int r = 0; r < B; ++r) {
    const int rows = (b.indptr[r + 1] - b.indptr[r]) * G;
    units[0] += (int64_t)hkv * ((rows + 15) / 16);
    units[1] += (int64_t)hkv * ((rows + 31) / 32);
  }
  const bool wide = units[1] >= 256;
  CHECK(p.rows_per_tile == (wide ? 32 : 16), "%d rows per tile", p.rows_per_tile);
  CHECK(p.units == units[wide] && p.row_groups == p.units, "units %lld", (long long)p.units);
  CHECK(p.padded_grid >= p.units && p.padded_grid % (kXcds * kXcdRun) == 0, "grid");
  CHECK(!p.needs_combine && p.ws_bytes == 0 && p.ws_o_bytes == 0 && p.ws_ml_bytes == 0, "workspace");
  for (int r = 0; r < B; ++r) {
    const int n = b.indptr[r + 1] - b.indptr[r];
    CHECK(prefix_chunks(b.plen[r], p.chunk_len[r]) == 1, "request %d is split", r);
    // and what the device rebuilds without a table
    CHECK(prefix_chunks(b.plen[r], chunk_keys(n, G, p.rows_per_tile, p.chunk_target, p.chunk_floor)) == 1, "request %d", r);
  }
  PlanTable t;
  fill_plan_table(t, B, b.indptr.data(), b.plen.data(), hkv, G, p);
  CHECK(t.count == (B > kPlanMax ? 0 : B) && t.merge_blocks == 0, "table");
  std::set<int> reqs;
  int64_t end = 0;
  for (int i = 0; i < t.count; ++i) {
    const PlanEntry &e = t.entry[i];
    const int r = plan_request(e.request_and_chunk);
    CHECK(r >= 0 && r < B && reqs.insert(r).second, "entry %d request %d", i, r);
    const int n = b.indptr[r + 1] - b.indptr[r];
    CHECK(plan_chunk_keys(e.request_and_chunk) == 0, "chunk of %d", r);   // the whole prefix
    CHECK(plan_nodes(e.n_and_len) == n && plan_prefix_len(e.n_and_len) == b.plen[r] && e.node_base == b.indptr[r],
          "sizes of %d", r);
    end += (int64_t)hkv * row_tiles(n, G, p.rows_per_tile);
    CHECK(e.unit_end == end && e.group_end == 0, "units of %d", r);
  }
}

static bool same_plan(const AttnPlan &x, const AttnPlan &y) {
  return x.rows_per_tile == y.rows_per_tile && x.chunk_target == y.chunk_target && x.chunk_floor == y.chunk_floor &&
         x.chunk_len == y.chunk_len && x.units == y.units && x.padded_grid == y.padded_grid &&
         x.row_groups == y.row_groups && x.needs_combine == y.needs_combine && x.single_tile == y.single_tile &&
         x.ws_o_bytes == y.ws_o_bytes &&
         x.ws_ml_bytes == y.ws_ml_bytes && x.ws_bytes == y.ws_bytes && x.est_us == y.est_us;
}

// The planner's choice against every choice of its two families, each made with
// integer divisions and priced in full: none is estimated much cheaper.  (The
// planner prices few of them in full, by lower bounds, and divides in floats.)
static int scratch_plans = 0;   // batches planned otherwise for the scratch

static void check_choice(const Batch &b, int hkv, int G, int D) {
  const int B = (int)b.plen.size();
  const int *ip = b.indptr.data(), *pl = b.plen.data();
  const AttnPlan p = make_plan(B, ip, pl, hkv, G, D, ADASERVE_BF16);
  CHECK(p.est_us == estimate_plan(B, ip, pl, hkv, G, D, p.chunk_len.data()), "estimate %g", p.est_us);
  double least = INFINITY;
  std::vector<int32_t> ck(B);
  auto price = [&]() { least = std::min(least, estimate_plan(B, ip, pl, hkv, G, D, ck.data())); };
  for (int fm : {8, 16, 32})
    for (int c = kMinChunk; c <= kMaxChunk; c *= 2) {
      for (int r = 0; r < B; ++r) ck[r] = chunk_keys(ip[r + 1] - ip[r], G, kMaxRowsPerTile, c, fm);
      price();
    }
  if (B <= kPlanMax) {
    int64_t work = 0;
    for (int r = 0; r < B; ++r)
      work += (int64_t)hkv * row_tiles(ip[r + 1] - ip[r], G, kMaxRowsPerTile) * std::max(1, ceil_div(pl[r], 32));
    for (int target : {160, 192, 224, 256, 288, 320, 352, 384, 416, 448, 512, 576, 640, 768, 1024}) {
      const int64_t per_unit = std::max<int64_t>(4, (work + target - 1) / target);
      for (int r = 0; r < B; ++r) {
        const int64_t blocks = ceil_div(pl[r], 32);
        const int64_t runs = std::max<int64_t>((blocks + per_unit - 1) / per_unit, (blocks + 255) / 256);
        ck[r] = blocks == 0 ? kMaxChunk : (int32_t)((blocks + runs - 1) / runs) * 32;
      }
      price();
    }
  }
  // within 10% for partials that fit the scratch, and within 10% for fewer units
  const bool fits = p.ws_bytes <= ADASERVE_TREE_ATTN_SCRATCH_BYTES;
  CHECK(p.est_us <= least * (fits ? 1.1 * 1.1 : 1.1) * (1 + 1e-12), "%g us, least %g", p.est_us, least);
  // in the scratch: the same plan if it fits, else one that does at a bearable
  // cost, else the same plan (which the call refuses)
  const AttnPlan s = make_plan(B, ip, pl, hkv, G, D, ADASERVE_BF16, true);
  const bool same = s.chunk_len == p.chunk_len && s.ws_bytes == p.ws_bytes;
  CHECK(same || (!fits && s.ws_bytes <= ADASERVE_TREE_ATTN_SCRATCH_BYTES && s.est_us <= least * 1.6 * 1.1 * (1 + 1e-12)),
        "in the scratch: %zu bytes, %g us, least %g", s.ws_bytes, s.est_us, least);
  scratch_plans += !same;
}

// One round of units, two per CU, unit by unit.
static void check_one_round(std::mt19937_64 &rng) {
  for (int it = 0; it < 400; ++it) {
    std::vector<UnitRun> runs;
    std::vector<UnitRun> each;
    const int most = 1 + (int)(rng() % 512);
    int total = 0, steps = 260;
    while (total < most) {
      steps = std::max(1, steps - (int)(rng() % 40));
      const int count = std::min(most - total, 1 + (int)(rng() % (it % 2 ? 300 : 12)));
      runs.push_back({steps, 1 + (int)(rng() % 4), 0.5 + (double)(rng() % 8) / 16, count});
      total += count;
      for (int i = 0; i < count; ++i) each.push_back(runs.back());
    }
    double worst = 0;
    for (int i = 0; i < std::min(total, 256); ++i)
      worst = std::max(worst, pair_us(each[i], i + 256 < total ? &each[i + 256] : nullptr));
    const UnitRun tiny{1, 1, 0.0, total};
    // what the starts add is the same for any units
    const double start = one_round_us({tiny}, total) - pair_us(tiny, total > 256 ? &tiny : nullptr);
    CHECK(std::fabs(one_round_us(runs, total) - start - worst) < 1e-9, "round of %d units", total);
  }
}

// The cached planner against a fresh plan on every call of a sequence that
// repeats batches, refills the same buffers in place (one prefix grows by a
// token, one tree loses a node) and changes only a scalar argument.
static void check_plan_cache(std::mt19937_64 &rng) {
  std::vector<int32_t> ip, pl;
  for (int it = 0; it < 400; ++it) {
    const int op = (int)(rng() % 5);
    if (ip.empty() || op == 0) {
      const Batch b = random_batch(rng, 1 + (int)(rng() % 40), 64, 20000);
      ip = b.indptr;
      pl = b.plen;
    } else if (op == 1) {
      pl[rng() % pl.size()] += 1;
    } else if (op == 2) {
      const size_t r = rng() % pl.size();
      if (ip[r + 1] - ip[r] > 1)
        for (size_t i = r + 1; i < ip.size(); ++i) ip[i] -= 1;
    }  // op 3, 4: the same contents again
    const int B = (int)pl.size();
    const int hkv = op == 4 ? 2 : 8, G = op == 4 ? 16 : 4, D = it % 2 ? 128 : 64;
    const AttnPlan fresh = make_plan(B, ip.data(), pl.data(), hkv, G, D, ADASERVE_BF16);
    const AttnPlan cached = make_plan_cached(B, ip.data(), pl.data(), hkv, G, D, ADASERVE_BF16);
    CHECK(same_plan(fresh, cached), "cached plan differs at step %d (op %d)", it, op);
    CHECK(same_plan(fresh, make_plan_cached(B, ip.data(), pl.data(), hkv, G, D, ADASERVE_BF16)),
          "second cached call differs at step %d", it);
  }
  CHECK(make_plan_cached(0, nullptr, nullptr, 8, 4, 128, ADASERVE_BF16).units == 0, "empty batch");
}

int main() {
  std::mt19937_64 rng(2501);
  // validation: malformed host mirrors and scalars give a status, never UB
  for (int it = 0; it < 20000; ++it) {
    const int B = (int)(rng() % 8);
    std::vector<int32_t> ip(B + 1), pl(B);
    for (auto &x : ip) x = (int32_t)(rng() % 3 == 0 ? rng() : rng() % 300) - (rng() % 7 == 0 ? 200 : 0);
    for (auto &x : pl) x = (int32_t)(rng() % 4 == 0 ? rng() : rng() % 40000) - (rng() % 9 == 0 ? 5 : 0);
    const int hq = (int)(rng() % 70) - 2, hkv = (int)(rng() % 20) - 2, D = rng() % 3 ? 128 : (int)(rng() % 300);
    AttnShape shape;
    const int32_t st = validate_attn_shape(B, ip.data(), pl.data(), hq, hkv, D, rng() % 5 ? 16 : 8,
                                           (int)(rng() % 3), (int)(rng() % 3000) - 1, shape);
    CHECK(st >= ADASERVE_OK && st <= ADASERVE_ERR_DEVICE, "status %d", st);
    CHECK(st != ADASERVE_OK || shape.total_nodes >= B, "accepted a batch with %d nodes", shape.total_nodes);
    if (st != ADASERVE_OK) CHECK(last_error_message()[0] != 0, "no message");
  }
  // planner on valid batches: small, named-workload-like and extreme shapes
  const int heads[][2] = {{32, 8}, {64, 8}, {8, 2}, {16, 16}, {32, 2}, {4, 2}, {16, 1}};
  for (int it = 0; it < 600; ++it) {
    const auto &h = heads[it % 7];
    const int B = 1 + (int)(rng() % (it % 5 == 0 ? 300 : 64));
    const Batch b = random_batch(rng, B, it % 3 ? 128 : 8, it % 4 ? 20000 : 200000);
    check_plan(b, h[0], h[1], it % 2 ? 128 : 64);
    check_f32_plan(b, h[0], h[1], it % 2 ? 128 : 64);
    if (it % 3 == 0) check_choice(b, h[1], h[0] / h[1], it % 2 ? 128 : 64);
  }
  {
    Batch b;  // the longest prefixes the validation accepts, the largest trees
    b.indptr = {0, 128, 256};
    b.plen = {kMaxPrefixLen, kMaxPrefixLen - 31};
    check_plan(b, 32, 2, 128);
    check_choice(b, 2, 16, 128);
    check_f32_plan(b, 32, 2, 128);
    check_plan(b, 128, 8, 64);
  }
  {
    Batch b;  // exactly kPlanMax requests and one more
    for (int extra = 0; extra < 2; ++extra) {
      b.indptr = {0};
      b.plen.clear();
      for (int r = 0; r < kPlanMax + extra; ++r) {
        b.indptr.push_back(b.indptr.back() + 1 + r % 128);
        b.plen.push_back(r * 97);
      }
      check_plan(b, 32, 8, 128);
      check_choice(b, 8, 4, 128);
      check_f32_plan(b, 32, 8, 128);
    }
  }
  check_plan_cache(rng);
  check_one_round(rng);
  {
    Batch b;  // in halves with a workspace, unsplit in the scratch
    b.indptr = {0};
    for (int r = 0; r < 65; ++r) b.indptr.push_back(b.indptr.back() + 5), b.plen.push_back(6630);
    const int before = scratch_plans;
    check_choice(b, 8, 8, 128);
    CHECK(scratch_plans == before + 1, "the same plan");
    // the two cache entries do not answer for each other
    const AttnPlan w = make_plan_cached(65, b.indptr.data(), b.plen.data(), 8, 8, 128, ADASERVE_BF16);
    const AttnPlan s = make_plan_cached(65, b.indptr.data(), b.plen.data(), 8, 8, 128, ADASERVE_BF16, true);
    CHECK(!same_plan(w, s), "cached plans");
    CHECK(same_plan(w, make_plan_cached(65, b.indptr.data(), b.plen.data(), 8, 8, 128, ADASERVE_BF16)), "cached plan");
  }
  // the makespan model against brute-force dealing
  for (int it = 0; it < 300; ++it) {
    std::vector<std::pair<double, int64_t>> u;
    const int k = 1 + (int)(rng() % 6);
    for (int i = 0; i < k; ++i) u.push_back({1.0 + (double)(rng() % 40), 1 + (int64_t)(rng() % 700)});
    auto copy = u;
    const double fast = lpt_makespan(copy);
    const double slow = brute_makespan(u, 512);
    CHECK(std::fabs(fast - slow) < 1e-9, "makespan %g vs %g", fast, slow);
  }
  std::printf("host plan checks passed: %d\n", g_checks);
  return 0;
}
