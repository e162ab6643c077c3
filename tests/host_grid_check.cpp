// The launch geometry that csrc/host.cpp computes for the kernels: no launch reaches 2^32 work-items in x (HIP's limit),
// and the launches of the one-body row kernel cover every tile of every row exactly once, each block on the XCD that
// the mapping names.
#include <algorithm>
#include <cstdio>
#include <utility>
#include <vector>

#include "host.h"

using namespace ffx;

static int fails = 0;
#define CHECK(c, ...)                  \
  do {                                 \
    if (!(c)) {                        \
      std::printf("FAIL: " __VA_ARGS__); \
      std::printf("\n");               \
      ++fails;                         \
    }                                  \
  } while (0)

static void onebody(int64_t rows, int64_t cols, int elem) {
  const OneBodyGrid g = onebody_grid(rows, cols, elem);
  CHECK(g.blocks < ((int64_t)1 << 32), "%lld x %lld: block numbers", (long long)rows, (long long)cols);
  std::vector<bool> seen((size_t)(g.row_blocks * g.tiles));
  for (int64_t b0 = 0; b0 < g.blocks; b0 += kOneBodyLaunch) {
    const int64_t n = std::min(g.blocks - b0, kOneBodyLaunch);
    CHECK(n * 256 < ((int64_t)1 << 32), "%lld x %lld: a launch of %lld blocks", (long long)rows, (long long)cols,
          (long long)n);
    CHECK(b0 % 8 == 0, "a launch starts within a round of XCDs");
    for (int64_t b = b0; b < b0 + n; ++b) {
      const OneBodyBlock ob = onebody_block((uint32_t)b, (uint32_t)g.row_blocks, g.per_xcd);
      if (g.per_xcd) CHECK(ob.tile % 8 == b % 8, "tile off its XCD");
      if (ob.tile >= g.tiles) continue;  // the kernel's own check
      const size_t at = (size_t)ob.tile * g.row_blocks + ob.row_block;
      CHECK(!seen[at], "a tile twice");
      seen[at] = true;
    }
  }
  size_t n = 0;
  for (bool x : seen) n += x;
  CHECK(n == seen.size(), "%lld x %lld: %zu of %zu tiles covered", (long long)rows, (long long)cols, n, seen.size());
}

int main() {
  // one row or column, ragged tiles, tiles per XCD and shared, one launch exactly full
  for (auto d : std::vector<std::pair<int64_t, int64_t>>{{1, 1}, {5, 63}, {3, 65}, {1287, 1287}, {1287, 449}, {12870, 12870},
                                                         {20, 38760}, {kOneBodyLaunch * 4, 64}, {kOneBodyLaunch * 4 + 1, 64}})
    for (int elem : {8, 16}) onebody(d.first, d.second, elem);
  // more than 2^32 amplitudes: 24 orbitals (6, 5), 32 orbitals (5, 4) and their mirrors
  onebody(binom(24, 6), binom(24, 5), 8);
  onebody(binom(32, 5), binom(32, 4), 8);
  onebody(binom(32, 4), binom(32, 5), 16);
  onebody(binom(32, 10), binom(32, 2), 8);
  // segment passes of long states: 29 orbitals (8, 3) in complex128, one block of 75 KB to a compute unit, and 31
  // orbitals (10, 2) in complex64 with the tables of complex rotations; 14 orbitals (7, 7) keep their 512 threads
  CHECK(seg_block_threads(60, 100 * 1024, binom(29, 8), 1, 256, 1024, 3654) * (binom(29, 8) + 7) < ((int64_t)1 << 32),
        "segment pass of 29 orbitals (8, 3)");
  CHECK(seg_block_threads(8, 31 * 1024, binom(31, 10), 1, 256, 1024, 465) * (binom(31, 10) + 7) < ((int64_t)1 << 32),
        "segment pass of 31 orbitals (10, 2)");
  CHECK(seg_block_threads(60, 70 * 1024, 3432, 1, 256, 1024, 3432) == 512, "segment pass of 14 orbitals (7, 7)");
  CHECK(seg_block_threads(1, 4096, binom(32, 16), 1, 256, 1024, 1) == 64, "one wave at the least");
  if (fails) return 1;
  std::printf("grid checks passed\n");
  return 0;
}
