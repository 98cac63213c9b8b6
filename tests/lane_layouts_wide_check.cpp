// Host-side check of the lane layouts at the wide blocks' thread counts (512,
// and 1024 in the finalize kernel), against the header the kernels include:
// the threads' cells cover the tile exactly once and their LDS words fall in
// distinct banks; the pair staging stages every cell and gives each one owner.
#include <cstdio>
#include <set>
#include <vector>

#include "bq_layout.hpp"

using namespace bqk;

static int failures = 0;
#define CHECK(c, ...)                  \
  do {                                 \
    if (!(c)) {                        \
      std::printf("FAIL: " __VA_ARGS__); \
      std::printf("\n");               \
      ++failures;                      \
    }                                  \
  } while (0)

template <typename T, int TY, int THREADS>
static void cells() {
  constexpr int CPT = TX * TY / THREADS;
  static_assert(CPT >= 1 && CPT * THREADS == TX * TY, "whole cells per thread");
  std::vector<int> seen(TX * TY, 0);
  std::vector<int> word[3];                   // per-cell reads of the radius-2 tile, the result rows, the corners
  const int pitch[3] = {32 * 3 + PITCH_MOD_TILE, 32 * 2 + PITCH_MOD_ROWS, 32 * 2 + PITCH_MOD_CORNERS};
  for (int t = 0; t < THREADS; ++t) {
    int vr = -1, vc = -1;
    cell_of<T, CPT>(t, vr, vc);
    const bool in = vr >= 0 && vr < TY && vc >= 0 && vc + CPT <= TX;
    CHECK(in, "tile of %d rows, %d threads: thread %d at (%d, %d)", TY, THREADS, t, vr, vc);
    if (!in) return;
    CHECK(vc % CPT == 0, "tile of %d rows, %d threads: thread %d not aligned to its vector", TY, THREADS, t);
    for (int k = 0; k < CPT; ++k) ++seen[vr * TX + vc + k];
    for (int p = 0; p < 3; ++p) word[p].push_back(vr * pitch[p] + vc);
  }
  for (int e = 0; e < TX * TY; ++e)
    CHECK(seen[e] == 1, "tile of %d rows, %d threads: cell %d taken %d times", TY, THREADS, e, seen[e]);
  if (sizeof(T) == 4)
    for (int p = 0; p < 3; ++p)
      for (int h = 0; h < THREADS; h += 32) {
        std::set<int> bank;
        for (int k = h; k < h + 32; ++k) bank.insert(word[p][k] % 32);
        CHECK(bank.size() == 32, "tile of %d rows, %d threads: pitch %d, half-wave %d in %zu banks", TY, THREADS,
              pitch[p], h / 32, bank.size());
      }
  std::printf("cells %zu-byte %d rows %d threads checked\n", sizeof(T), TY, THREADS);
}

template <int NPR, int NR, int THREADS>
static void staging() {
  using S = PairStaging<NPR, NR, THREADS>;
  std::vector<int> staged(NR * 2 * NPR, 0), owned(NR * 2 * NPR, 0);
  for (int t = 0; t < THREADS; ++t)
    for (int k = 0; k < S::K; ++k) {
      const int r = S::row(t, k), c = S::col(t);
      const bool in = r >= 0 && r < NR && c >= 0 && c + 1 < 2 * NPR;
      CHECK(in, "%d x %d, %d threads: thread %d round %d at (%d, %d)", NR, 2 * NPR, THREADS, t, k, r, c);
      if (!in) continue;
      for (int u = 0; u < 2; ++u) {
        ++staged[r * 2 * NPR + c + u];
        if (S::owns(t, k)) ++owned[r * 2 * NPR + c + u];
      }
    }
  for (int e = 0; e < NR * 2 * NPR; ++e)
    CHECK(staged[e] >= 1 && owned[e] == 1, "%d x %d, %d threads: cell %d staged %d times, owned %d times", NR, 2 * NPR,
          THREADS, e, staged[e], owned[e]);
  std::printf("staging %d x %d %d threads checked\n", NR, 2 * NPR, THREADS);
}

// the stencil kernel's radius-2, radius-1 and corner rows, the finalize
// kernel's corner rows
template <int TY, int THREADS>
static void tile() {
  staging<(TX + 4) / 2, TY + 4, THREADS>();
  staging<(TX + 4) / 2, TY + 2, THREADS>();
  staging<(TX + 6) / 2, TY + 5, THREADS>();
  staging<(TX + 4) / 2, TY + 3, THREADS>();
}

int main() {
  cells<float, 16, 512>();
  cells<float, 16, 1024>();
  cells<float, 8, 512>();
  cells<double, 8, 512>();
  tile<16, 512>();
  tile<16, 1024>();
  tile<8, 512>();
  if (failures) std::printf("%d failures\n", failures);
  return failures ? 1 : 0;
}
