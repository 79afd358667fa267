// CPU test of stage-batched layouts in which cells launch nothing at some steps (a null
// variant): every recorded launch in exactly one launch of its step, branch and variant,
// an empty step in none, and the cells' order turning at each step that launches anything.
#include <cstdio>
#include <random>
#include <set>
#include <tuple>
#include <vector>

#include "queue_layout.h"

using namespace fhe;

static int failures = 0;
#define CHECK(c)                                                  \
  do {                                                            \
    if (!(c)) {                                                   \
      std::printf("FAIL %s:%d: %s\n", __FILE__, __LINE__, #c);    \
      ++failures;                                                 \
    }                                                             \
  } while (0)

int main() {
  static const int variants[3] = {0, 0, 0};
  std::mt19937 rng(11);
  for (int trial = 0; trial < 300; ++trial) {
    const int nc = 1 + (int)(rng() % 12), ns = 9, nbr = 1 + (int)(rng() % 3);
    // steps at which every cell, some cells or no cell launches nothing
    int mode[ns];
    for (int& m : mode) m = (int)(rng() % 4);
    std::vector<std::vector<QRec>> recs(nc, std::vector<QRec>(ns));
    std::set<std::tuple<int, int, const void*>> keys;
    for (int c = 0; c < nc; ++c) {
      const int br = (int)(rng() % nbr);
      for (int s = 0; s < ns; ++s) {
        QRec& r = recs[c][s];
        r.branch = br;
        if (mode[s] == 0 || (mode[s] == 1 && rng() % 2)) continue;  // nothing at this step
        const int v = (int)(rng() % 3);
        r.variant = &variants[v];
        r.bx = v == 2 ? 256 : 128;
        r.by = r.bz = r.gz = 1;
        r.gx = 1 + (uint32_t)(rng() % 40);
        r.gy = 1 + (uint32_t)(rng() % 3);
        r.arg_bytes = 64 * (1 + v);
        keys.insert(std::make_tuple(s, br, r.variant));
      }
    }
    std::vector<QLaunch> lay;
    CHECK(queue_layout(recs, &lay) == QL_OK);
    CHECK(lay.size() == keys.size());
    std::vector<std::vector<int>> seen(nc, std::vector<int>(ns, 0));
    int step = -1, turns = -1;
    for (const QLaunch& L : lay) {
      CHECK(L.step >= step && L.variant && !L.segs.empty());
      if (L.step != step) ++turns;
      step = L.step;
      uint32_t end = 0;
      for (size_t i = 0; i < L.segs.size(); ++i) {
        const QSeg& g = L.segs[i];
        const QRec& r = recs[g.cell][L.step];
        CHECK(g.off == end && g.gx == r.gx && g.gy == r.gy);
        CHECK(r.branch == L.branch && r.variant == L.variant);
        if (i > 0) CHECK((turns & 1) ? g.cell < L.segs[i - 1].cell : g.cell > L.segs[i - 1].cell);
        end = g.off + ((g.gx * g.gy + 7) & ~7u);
        ++seen[g.cell][L.step];
      }
      CHECK(L.blocks == end);
    }
    for (int c = 0; c < nc; ++c)
      for (int s = 0; s < ns; ++s) CHECK(seen[c][s] == (recs[c][s].variant ? 1 : 0));
  }
  // one cell with its two stages in one kernel, one with a launch for each
  {
    std::vector<std::vector<QRec>> recs(2, std::vector<QRec>(3));
    for (auto& cell : recs)
      for (auto& r : cell) {
        r.variant = &variants[0];
        r.gx = r.gy = r.gz = 1;
        r.arg_bytes = 8;
      }
    recs[0][1] = QRec{};
    std::vector<QLaunch> lay;
    CHECK(queue_layout(recs, &lay) == QL_OK);
    CHECK(lay.size() == 3 && lay[0].segs.size() == 2 && lay[1].segs.size() == 1 && lay[1].segs[0].cell == 1 &&
          lay[2].segs.size() == 2);
  }
  if (failures) {
    std::printf("%d FAILURES\n", failures);
    return 1;
  }
  std::printf("ALL PASSED\n");
  return 0;
}
