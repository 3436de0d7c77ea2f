// Host check of the page write's item arithmetic (no GPU): whatever row the search over
// cu_new returns, a page item is inactive or writes a page of that row's block table; and
// for non-decreasing cu_new, also one that starts past 0, every token has exactly one item.
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "ra_page_write.h"

using ra::pwrite::WriteArgs;
using ra::pwrite::WriteItem;

static int failures = 0;

static void check(const std::vector<int> &cu, const std::vector<int> &start, int total, int max_new,
                  int max_pos, bool valid) {
  const int B = (int)start.size(), stride = (max_pos + 15) / 16, pages = 7;
  constexpr int kMargin = 1 << 16;   // an index outside the table reads this host memory instead
  std::vector<int> table(2 * kMargin + (size_t)B * stride, 3);
  WriteArgs a{};
  a.cu_new = cu.data(), a.start_pos = start.data();
  a.block_table = table.data() + kMargin;
  a.bt_stride = stride, a.num_pages = pages, a.hkv = 1;
  a.total_new = total, a.max_new = max_new, a.max_pos = max_pos;
  std::vector<int> covered(total, 0);
  const int64_t items = ra::pwrite::write_items(B, total);
  for (int item = 0; item < items; ++item) {
    // the row the kernel's search finds, its 64 probes a round counted here
    const int found = ra::search_rounds(B, [&](int lo, int step, int len) {
      int hits = 0;
      for (int off = 0; off < 64 * step && off < len; off += step) {
        if (lo + off < 0 || lo + off >= B) {
          ++failures;
          std::printf("probe of row %d of %d\n", lo + off, B);
          std::exit(1);
        }
        hits += ra::pwrite::row_item(a, lo + off) <= item;
      }
      return hits;
    });
    if (valid) {
      int last = 0;
      for (int b = 0; b < B; ++b)
        if (ra::pwrite::row_item(a, b) <= item) last = b;
      if (found != last && failures++ < 5) std::printf("item %d: row %d, not %d\n", item, found, last);
    }
    for (int b = 0; b < B; ++b) {
      const int chunk = item - ra::pwrite::row_item(a, b);
      if (chunk < -kMargin / 2) continue;
      const WriteItem it = ra::pwrite::write_item(a, chunk, b);
      if (!it.active) continue;
      const int64_t n = it.hi - it.lo, src = it.cu0 + it.lo - it.s;
      if (it.pg < 0 || it.pg >= stride || n <= 0 || src < 0 || src + n > total) {
        if (failures++ < 5)
          std::printf("row %d chunk %d: page %d of %d, tokens %lld + %lld of %d\n", b, chunk, it.pg,
                      stride, (long long)src, (long long)n, total);
      }
    }
    const WriteItem it = ra::pwrite::write_item(a, item - ra::pwrite::row_item(a, found), found);
    if (it.active)
      for (int p = it.lo; p < it.hi; ++p) {
        const int src = it.cu0 + p - it.s;
        if (src >= 0 && src < total) ++covered[src];
      }
  }
  if (!valid) return;
  for (int t = 0; t < total; ++t)
    if (covered[t] != (t >= cu[0] && t < cu[B])) {
      if (failures++ < 5) std::printf("token %d of [%d, %d): %d items\n", t, cu[0], cu[B], covered[t]);
    }
}

int main() {
  std::mt19937 rng(5);
  auto pick = [&](int lo, int hi) { return lo + (int)(rng() % (unsigned)(hi - lo + 1)); };
  for (int round = 0; round < 400; ++round) {
    const int B = round % 40 == 7 ? pick(60, 300) : pick(1, 12), longest = pick(1, 90);
    std::vector<int> cu(B + 1), start(B);
    cu[0] = round % 2 ? pick(0, 200) : 0;   // a slice of a longer cu_new
    int last = 0;
    for (int b = 0; b < B; ++b) {
      cu[b + 1] = cu[b] + pick(0, longest);
      start[b] = pick(0, 100);
      last = std::max(last, start[b] + cu[b + 1] - cu[b]);
    }
    check(cu, start, cu[B] + pick(0, 20), longest, last + pick(0, 20), true);
    for (int b = 0; b <= B; ++b) cu[b] = pick(-50, 300);   // any order
    for (int b = 0; b < B; ++b) start[b] = pick(-20, 200);
    check(cu, start, pick(1, 250), pick(1, 90), pick(1, 180), false);
  }
  std::printf("%d failures\n", failures);
  return failures != 0;
}
