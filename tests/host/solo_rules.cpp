// Rules of the single-workgroup launches and of the batch's directions that can
// be checked without a GPU.
// Prints "ok" and exits 0 when every check holds.
#include <algorithm>
#include <cstdio>

#include "../../paper_1708_01159_amd/csrc/gsw_internal.h"

using namespace gsw;

#define CHECK(c)                                                          \
  do {                                                                    \
    if (!(c)) {                                                           \
      std::fprintf(stderr, "check failed: %s (line %d)\n", #c, __LINE__); \
      return 1;                                                           \
    }                                                                     \
  } while (0)

int main() {
  // A row of a level that a launch takes is walked over exactly its arcs: at
  // most kSoloMaxArcs in all by the largest degree or by a count, kSoloHubMax
  // where a few rows hold most of them, any number up to kSoloWholeArcs on a graph
  // searched to the end.
  int64_t most = kSoloMaxArcs > kSoloWholeArcs ? kSoloMaxArcs : kSoloWholeArcs;
  if (kSoloHubMax > most) most = kSoloHubMax;
  for (int64_t deg = 0; deg <= most; ++deg) {
    if (solo_row_length(deg) != deg) std::fprintf(stderr, "row of %lld arcs\n", (long long)deg);
    CHECK(solo_row_length(deg) == deg);
  }
  for (int k = 0; k < GSW_N_KERNELS; ++k)
    for (int32_t nf = 1; nf <= kSoloMax; ++nf) {
      CHECK(solo_arc_limit(k, nf) <= kSoloMaxArcs);
      CHECK(!solo_takes(k, nf, most + 1, most + 1));
    }
  // a hub's row, or a few in a row, that the level kernel would leave to one
  // workgroup, but not where its arcs are spread over the grid
  for (int64_t arcs : {kSoloHubMin, (int64_t)16000, (int64_t)49998, kSoloHubMax}) {
    CHECK(solo_takes(GSW_K_PUSH_VERTEX, 1, arcs, arcs) && solo_takes(GSW_K_PUSH_WAVE16, 300, arcs, arcs * 2 / 3));
    CHECK(!solo_takes(GSW_K_PUSH_VERTEX, 300, arcs, arcs / 2) && !solo_takes(GSW_K_PUSH_EDGE, 1, arcs, arcs));
  }
  // a longer row's level is handed back, by its counted arcs and not by this
  // length, which must still be one that no sum is taken of
  const int64_t lens[] = {most + 1, 0x7ffffffell, 0x7fffffffll, 0x80000000ll, 0x100000000ll, 0x7fffffffffll};
  for (int64_t deg : lens) CHECK(solo_row_length(deg) > kSoloMaxArcs);
  // Batched sources go bottom-up together by a rule of its own: it does not
  // follow a push_to_pull below the default down, and one that never pulls
  // keeps it from doing so.
  for (float f : {0.0f, 0.0001f, 0.003f, 0.01f, 0.03f, 0.0699f}) CHECK(ms_together(f) >= 0.5 * (double)kMsPushToPull);
  for (float f : {kMsPushToPull, 0.1f, 0.2f, 1.0f, 1e9f}) CHECK(ms_together(f) == 0.5 * (double)f);
  // Hub rows of a batch: by one wave only for one or two sources that pull by
  // their own frontiers.
  for (int pulling = 0; pulling <= 64; ++pulling) {
    CHECK(ms_hub_chunks(1, pulling, true) && ms_hub_chunks(2, pulling, false));
    CHECK(ms_hub_chunks(1, pulling, false) == (pulling > 2));
  }
  std::puts("ok");
  return 0;
}
