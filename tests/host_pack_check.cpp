// The device forms of the segment class tables (csrc/host.cpp: compact_members, split_seg_window,
// pack_class_codes) against the tables they are made from: every class of every window must reach the same
// members, in the same order.
#include <cstdio>
#include <cstdlib>
#include <set>
#include <vector>

#include "host.h"

using namespace ffx;

static int fails = 0;
#define CHECK(c, ...)              \
  do {                             \
    if (!(c)) {                    \
      std::printf("FAIL: " __VA_ARGS__); \
      std::printf("\n");           \
      ++fails;                     \
    }                              \
  } while (0)

using Members = std::multiset<std::vector<int>>;

static Members from_table(const SegWindowTable& t, int w) {
  Members s;
  for (size_t ch = 0; ch < t.chunk_m.size(); ++ch)
    for (int j = 0; j < 64; ++j) {
      const int c = t.code[ch * 64 + j];
      if (c < 0) continue;
      const int m = t.chunk_m[ch];
      std::vector<int> v;
      for (int k = 0; k < (int)binom(w, m); ++k) v.push_back((c >> 5) + t.mt[t.mt[m * t.nl1 + (c & 31)] + k]);
      s.insert(v);
    }
  return s;
}

// members as the kernels address them: base (in units of the lane's element) + stride * 16-bit offset
static Members from_device(const SegWindowTable& t, const std::vector<uint16_t>& off, int w, int stride) {
  Members s;
  const std::vector<int> codes = pack_class_codes(t, 0);
  for (size_t ch = 0; ch < t.chunk_m.size(); ++ch)
    for (int j = 0; j < 64; ++j) {
      const int c = codes[ch * 64 + j];
      if (c < 0) continue;
      const size_t word = (size_t)(c & ((1 << kCodeMoffBits) - 1));
      const int n = (int)binom(w, t.chunk_m[ch]);
      CHECK((word + (n + 7) / 8) * 8 <= off.size(), "table words past the end");
      std::vector<int> v;
      for (int k = 0; k < n; ++k) v.push_back((c >> kCodeMoffBits) + stride * (int)off[word * 8 + k]);
      s.insert(v);
    }
  return s;
}

int main() {
  const int sectors[][2] = {{6, 3}, {7, 1}, {8, 4}, {9, 8}, {10, 5}, {12, 6}, {13, 2}, {14, 7}, {16, 8}, {20, 2}};
  for (const auto& ne : sectors) {
    const int N = ne[0], n = ne[1], w = 6;
    for (int wt : {N, N - 1}) {
      if (wt < w) continue;
      const auto strs = make_strings(N, n);
      for (const auto& run : segment_runs(strs, wt)) {
        const std::vector<uint64_t> seg(strs.begin() + run.first, strs.begin() + run.first + run.second);
        std::vector<uint16_t> off, off2;
        for (int a = 0; a + w <= wt; ++a) {
          SegWindowTable t = build_seg_window(seg, wt, a, w, 8);
          const Members want = from_table(t, w);
          SegWindowTable sp = split_seg_window(t, w);
          balance_seg_window(t, w, 12);
          CHECK(from_device(compact_members(t, w, off), off, w, 1) == want, "N=%d n=%d a=%d compact", N, n, a);
          Members parts;
          for (const auto& v : want)
            for (int part = 0; part < 2; ++part) {
              std::vector<int> q;
              for (int x : v) q.push_back(2 * x + part);
              parts.insert(q);
            }
          balance_seg_window(sp, w, 8);
          const SegWindowTable dsp = compact_members(sp, w, off2);
          CHECK(from_device(dsp, off2, w, 2) == parts, "N=%d n=%d a=%d split", N, n, a);
          // the two parts of a class sit in neighbouring lanes
          for (size_t i = 0; i + 1 < dsp.code.size(); i += 2)
            CHECK(dsp.code[i] < 0 ? dsp.code[i + 1] < 0 : dsp.code[i + 1] == dsp.code[i] + 32, "lane pair");
        }
        CHECK(off == off2, "the two forms share their member tables");
      }
    }
  }
  if (fails) return 1;
  std::printf("pack checks passed\n");
  return 0;
}
