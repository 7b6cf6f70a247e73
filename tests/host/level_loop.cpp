// The host's level loop against a replay of the device's control protocol:
// every search ends with all its levels read, whatever mix of level-kernel and
// single-workgroup launches the loop has queued when a level needs two
// launches or is handed back, and no record is overwritten before it is read.
// Prints "ok" and exits 0 when every search does.
#include <algorithm>
#include <random>

#include "fake_hip.h"

using namespace gsw;

namespace {

struct Case {
  const char* name;
  int64_t n, nnz, deg_max;
  fake::Script script;
  std::vector<int32_t> sched;  // kernels by depth (one: fixed)
  bool count_arcs = false, hubs = false, symmetric = true;
};

int64_t g_levels = 0, g_solo = 0, g_back = 0, g_runs = 0;

bool run(const Case& c) {
  gsw_graph g;
  g.n = c.n;
  g.nnz = c.nnz;
  g.symmetric = c.symmetric ? 1 : 0;
  g.deg_stats[4] = (double)c.deg_max;
  Workspace w;
  w.n = c.n;
  w.nw = (c.n + 63) / 64;
  std::vector<unsigned long long> ring((size_t)kBfsRing * kBfsRec);
  BfsCtl ctl[2] = {};
  w.ring = w.d_ring = ring.data();
  w.ctl = ctl;
  std::vector<int32_t> sched = c.sched;
  w.d_sched = sched.data();
  gsw_bfs_opts o;
  gsw_bfs_opts_default(&o);
  o.policy = sched.size() == 1 ? GSW_POLICY_FIXED : GSW_POLICY_SCHEDULE;
  o.fixed_kernel = sched[0];
  o.schedule = sched.data();
  o.schedule_len = (int32_t)sched.size();
  o.count_arcs = c.count_arcs ? 1 : 0;
  const BfsPolicy dp = device_policy(&g, w, &o, true, true);
  const SearchPolicy pol{&o, true, true, c.hubs};
  const size_t depth = c.script.nf.size();
  std::vector<gsw_level_trace> trace(depth);
  int32_t rows = 0;
  fake::dev = fake::Device();
  fake::dev.script = c.script;
  fake::dev.rows = &rows;
  const gsw_status st = run_levels(&g, w, nullptr, pol, dp, 0, 0, nullptr, nullptr, trace.data(), (int32_t)depth,
                                   &rows, nullptr);
  ++g_runs;
  g_levels += rows;
  g_solo += fake::dev.solo_levels;
  g_back += fake::dev.handed_back;
  bool ok = st == GSW_OK && !fake::dev.stalled && !fake::dev.overrun && rows == (int32_t)depth;
  for (size_t d = 0; ok && d < depth; ++d)
    ok = trace[d].n_frontier == c.script.nf[d] &&
         trace[d].kernel == c.sched[std::min(d, c.sched.size() - 1)];
  if (!ok) {
    std::fprintf(stderr, "%s: n %lld, arcs %lld, largest degree %lld: status %d, %d of %zu levels read%s%s; kernels",
                 c.name, (long long)c.n, (long long)c.nnz, (long long)c.deg_max, (int)st, rows, depth,
                 fake::dev.stalled ? ", stalled" : "", fake::dev.overrun ? ", record overwritten" : "");
    for (size_t d = 0; d < c.sched.size() && d < 12; ++d) std::fprintf(stderr, " %d", c.sched[d]);
    std::fprintf(stderr, "; frontiers");
    for (int32_t d = std::max(0, rows - 6); d < (int32_t)depth && d < rows + 6; ++d)
      std::fprintf(stderr, " %d", c.script.nf[(size_t)d]);
    std::fprintf(stderr, "\n");
  }
  return ok;
}

fake::Script layers(std::vector<int32_t> nf, int64_t degree) {
  fake::Script s;
  s.nf = std::move(nf);
  for (int32_t x : s.nf) s.arcs.push_back(x * degree);
  return s;
}

Case random_case(std::mt19937_64& rng) {
  auto pick = [&](std::vector<int64_t> v) { return v[rng() % v.size()]; };
  Case c;
  c.name = "random";
  // on both sides of a whole graph, of the small bitmap and of the one that LDS holds
  c.n = pick({1500, 2048, 2049, 30000, 131072, 131073, 900000, 1048576, 1048577, 4000000});
  c.deg_max = pick({2, 4, 5, 8, 16, 40, 513, 5000, 100000});
  c.nnz = std::max<int64_t>(2 * c.deg_max, c.n * pick({1, 2, 8, 16, 32}));
  if (c.n <= kSoloMax && rng() % 2) c.nnz = std::min<int64_t>(c.nnz, kSoloWholeArcs);
  c.count_arcs = rng() % 3 == 0;
  c.symmetric = rng() % 4 != 0;
  c.hubs = rng() % 8 == 0;
  // frontiers that stay at, below or beyond the sizes at which rules change
  const int64_t depth = pick({1, 3, 8, 30, 60, 150, 700});
  int64_t left = c.n - 1, size = 1;
  for (int64_t d = 0; d < depth && size > 0; ++d) {
    c.script.nf.push_back((int32_t)size);
    const int64_t per = 1 + (int64_t)(rng() % (uint64_t)std::min<int64_t>(c.deg_max, 64));
    c.script.arcs.push_back(std::min<int64_t>(size * c.deg_max, std::max<int64_t>(size * per, 1)));
    int64_t next;
    switch (rng() % 6) {
      case 0: next = size + (int64_t)(rng() % 3) - 1; break;
      case 1: next = pick({500, 512, 513, 800, 1000, 1024, 1025, 1500, 2048, 2049, 3000}); break;
      case 2: next = size - (int64_t)(rng() % 50); break;
      case 3: next = (int64_t)(rng() % 60) + 1; break;
      case 4: next = size * 2; break;
      default: next = size; break;
    }
    size = std::min<int64_t>(std::max<int64_t>(next, 1), left);
    left -= size;
  }
  const int push[] = {GSW_K_PUSH_VERTEX, GSW_K_PUSH_WAVE8, GSW_K_PUSH_EDGE, GSW_K_PUSH_EDGE};
  const int any[] = {GSW_K_PUSH_EDGE, GSW_K_PUSH_EDGE, GSW_K_PUSH_VERTEX, GSW_K_PULL_BITMAP, GSW_K_VERTEX_SCAN};
  switch (rng() % 3) {
    case 0: c.sched = {GSW_K_PUSH_EDGE}; break;
    case 1:
      for (size_t d = 0; d < c.script.nf.size(); ++d) c.sched.push_back(push[rng() % 4]);
      break;
    default:
      for (size_t d = 0; d < c.script.nf.size(); ++d) c.sched.push_back(any[rng() % 5]);
      break;
  }
  return c;
}

}  // namespace

int main() {
  int bad = 0;
  const std::vector<int32_t> edge = {GSW_K_PUSH_EDGE};
  std::vector<int32_t> wide = {1, 16, 200};
  wide.insert(wide.end(), 30, 800);
  std::vector<int32_t> deep(40, 3);
  deep[0] = 1;
  deep.insert(deep.end(), 30, 1500);
  std::vector<int32_t> mid = {1, 40, 300};
  mid.insert(mid.end(), 30, 600);
  std::vector<Case> cases = {
      {"800 a level", 30000, 480000, 16, layers(wide, 16), edge},
      {"shrinking tail", 200000, 3200000, 16, layers({1, 16, 250, 3000, 20000, 950, 700, 300, 60, 4}, 16), edge},
      {"600 a level, 40 arcs a row", 30000, 1200000, 40, layers(mid, 40), edge},
      {"1500 a level past depth 32", 200000, 3200000, 16, layers(deep, 16), edge},
      {"whole graph, scans first", 2000, 20000, 40, layers({1, 20, 700, 600}, 8),
       {GSW_K_VERTEX_SCAN, GSW_K_PUSH_VERTEX, GSW_K_PUSH_EDGE, GSW_K_PUSH_EDGE}},
  };
  for (int64_t n : {200000, 4000000})
    for (int32_t width : {1, 500, 1500}) {
      std::vector<int32_t> flat((size_t)std::min<int64_t>(3000, n / width - 1), width);
      flat[0] = 1;
      cases.push_back({"long and even", n, 4 * n, 4, layers(flat, 4), edge});
    }
  std::vector<int32_t> doubled(34, 4);  // 2048, taken, then 4096, which pending launches pass on
  doubled[0] = 1;
  doubled.insert(doubled.end(), {2049, 4096, 2048, 4096, 30, 10});
  cases.push_back({"doubled past depth 32", 900000, 3600000, 4, layers(doubled, 3), edge});
  // Levels that are handed back one after another: few launches in vain, and
  // short levels behind one are taken again.
  std::vector<int32_t> even(400, 1500), hubs(400, 1);
  even[0] = 1;
  for (int k : {GSW_K_PUSH_EDGE, GSW_K_PUSH_WAVE4}) {
    Case c{"1500 a level, 24 arcs a row", 700000, 16800000, 30, layers(even, 24), {k}};
    Case h{"a path with hubs", 700000, 16800000, 100000, layers(hubs, 3), {k}};
    for (size_t d = 5; d < hubs.size(); d += 40) h.script.arcs[d] = 100000;
    c.n = 60000;
    if (!run(c)) return 1;
    const int64_t back = fake::dev.handed_back;
    if (!run(h)) return 1;
    if (back > 40 || fake::dev.solo_levels < 300) {
      std::fprintf(stderr, "%lld of 400 even levels handed back; %lld of 400 on a path taken\n", (long long)back,
                   (long long)fake::dev.solo_levels);
      return 1;
    }
  }
  std::mt19937_64 rng(20);
  for (int i = 0; i < 60000; ++i) cases.push_back(random_case(rng));
  for (const Case& c : cases)
    if (!run(c) && ++bad >= 12) break;
  if (bad) return 1;
  if (g_solo < g_levels / 10 || g_back < 1000) {
    std::fprintf(stderr, "too few single-workgroup levels: %lld of %lld, %lld handed back\n", (long long)g_solo,
                 (long long)g_levels, (long long)g_back);
    return 1;
  }
  std::puts("ok");
  return 0;
}
