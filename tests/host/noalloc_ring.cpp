// The mapped host memory that gsw_bfs_noalloc's level records go to, without a
// GPU: graphs are made whether or not there is any, searches end with and
// without it, all graphs share it, and the last one gives it back.
// Prints "ok" and exits 0 when every check holds.
#include "fake_hip.h"

using namespace gsw;

#define CHECK(c)                                                                                    \
  do {                                                                                              \
    if (!(c)) {                                                                                     \
      std::fprintf(stderr, "check failed: %s (line %d): %s\n", #c, __LINE__, gsw_last_error());     \
      std::exit(1);                                                                                 \
    }                                                                                               \
  } while (0)

namespace {

gsw_graph* path(int64_t n) {
  std::vector<int64_t> offs((size_t)n + 1, 0);
  std::vector<int32_t> cols;
  for (int64_t v = 0; v < n; ++v) {
    if (v > 0) cols.push_back((int32_t)(v - 1));
    if (v + 1 < n) cols.push_back((int32_t)(v + 1));
    offs[(size_t)v + 1] = (int64_t)cols.size();
  }
  gsw_graph* g = nullptr;
  CHECK(gsw_graph_create_host(n, (int64_t)cols.size(), offs.data(), cols.data(), GSW_ASSUME_SYMMETRIC, &g) == GSW_OK);
  return g;
}

// A search of `depth` levels from each of three sources, by push_edge, single-
// workgroup launches among them or not.
void search(gsw_graph* g, int32_t depth, int32_t width, bool solo) {
  fake::dev = fake::Device();
  fake::dev.script.nf.assign((size_t)depth, width);
  fake::dev.script.nf[0] = 1;
  for (int32_t x : fake::dev.script.nf) fake::dev.script.arcs.push_back(2 * x);
  gsw_bfs_opts o;
  gsw_bfs_opts_default(&o);
  o.policy = GSW_POLICY_FIXED;
  o.fixed_kernel = GSW_K_PUSH_EDGE;
  o.device_ptrs = 1;
  o.no_solo = solo ? 0 : 1;
  const int32_t src[3] = {0, 1, 2};
  std::vector<int32_t> levels(3 * (size_t)g->n);
  std::vector<gsw_level_trace> trace(3 * (size_t)depth);
  int32_t rows = 0;
  CHECK(gsw_bfs_noalloc(g, src, 3, levels.data(), nullptr, trace.data(), 3 * depth, &rows, &o) == GSW_OK);
  CHECK(rows == 3 * depth && !fake::dev.stalled);
  for (int32_t i = 0; i < rows; ++i)
    CHECK(trace[(size_t)i].source_idx == i / depth && trace[(size_t)i].level == i % depth &&
          trace[(size_t)i].n_frontier == fake::dev.script.nf[(size_t)(i % depth)]);
  CHECK((fake::dev.solo_levels > 0) == solo);
}

void searches(gsw_graph* g) {
  for (int32_t width : {1, 600, 3000})
    for (int32_t depth : {1, 2, 9, 300, 1000}) {
      if ((int64_t)width * depth >= g->n) continue;
      search(g, depth, width, true);
      search(g, depth, width, false);
    }
}

}  // namespace

int main() {
  const int64_t most = GSW_NOALLOC_MAX_VERTICES;
  for (int64_t n : {(int64_t)5000, most, most + 1}) {  // mapped memory: as usual
    gsw_graph* g = path(n);
    if (n <= most) searches(g);
    gsw_graph_destroy(g);
  }
  CHECK(fake::pinned == 0);
  fake::pinned_room = 0;  // none to be had: graphs are made, and search as well
  {
    gsw_graph* g = path(200000);
    searches(g);
    fake::pinned_room = 1 << 20;  // ... and a graph made later has it
    gsw_graph* h = path(200000);
    searches(h);
    searches(g);
    gsw_graph_destroy(h);
    searches(g);
    gsw_graph_destroy(g);
  }
  CHECK(fake::pinned == 0);
  fake::pinned_room = (size_t)1 << 40;
  std::vector<gsw_graph*> many;
  for (int i = 0; i < 50; ++i) many.push_back(path(3000));
  const size_t ring = (size_t)kBfsRing * kBfsRec * sizeof(unsigned long long);
  CHECK(fake::pinned <= ring);  // one for all
  for (size_t i = 0; i < many.size(); ++i) {
    gsw_graph_destroy(many[i]);
    if (i + 1 < many.size()) search(many.back(), 9, 20, true);
  }
  CHECK(fake::pinned == 0);
  std::puts("ok");
  return 0;
}
