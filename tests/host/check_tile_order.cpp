// Host check of the attention kernels' tile order (common.h): every tile once,
// and no XCD left with much more work than the others, for list offsets of
// heads that are alike and of heads that are not.
#include <algorithm>
#include <cstdio>
#include <vector>

#include "common.h"

namespace {
int failures = 0;

// work[h]: list entries per tile of head h
void check(const char* name, unsigned nblk, const std::vector<int>& work, bool want_by_head) {
  std::vector<int32_t> ptr = {0};
  for (int per : work)
    for (unsigned t = 0; t < nblk; ++t) ptr.push_back(ptr.back() + per);
  const unsigned tiles = (unsigned)work.size() * nblk;
  std::vector<int> seen(tiles, 0);
  int64_t load[8] = {};
  bool by_head = true;
  for (unsigned wg = 0; wg < tiles; ++wg) {
    const unsigned first = ut::group_tile(wg / nblk, nblk);
    const bool alike = ut::heads_alike([&](int x) { return ptr[first + x * nblk]; });
    by_head = by_head && alike;
    const unsigned lt = alike ? ut::head_tile(wg, first, nblk) : wg;
    if (lt < tiles) ++seen[lt];
    if (lt < tiles) load[wg & 7] += ptr[lt + 1] - ptr[lt];
    if (alike && lt / nblk % 8 != wg % 8) ++failures;   // whole heads per XCD
  }
  const bool once = std::all_of(seen.begin(), seen.end(), [](int n) { return n == 1; });
  // plain order deals tiles out singly: one tile of each head more at most
  int64_t slack = 0;
  for (int per : work) slack += per;
  const int64_t most = *std::max_element(load, load + 8);
  const bool even = most <= ptr.back() / 8 + ptr.back() / 256 + slack;
  const bool ok = once && even && by_head == want_by_head;
  std::printf("%-36s %s (longest XCD %lld of %d entries)\n", name, ok ? "ok" : "FAIL", (long long)most,
              ptr.back());
  if (!ok) ++failures;
}
}  // namespace

int main() {
  check("equal heads", 52, std::vector<int>(24, 16), true);
  check("one block per head", 1, std::vector<int>(8, 1), true);
  check("empty lists", 7, std::vector<int>(8, 0), true);
  check("within the margin", 100, {100, 100, 102, 100, 100, 100, 99, 100}, true);
  check("past the margin", 100, {100, 100, 110, 100, 100, 100, 99, 100}, false);
  check("one dense head of eight", 52, {52, 3, 3, 3, 3, 3, 3, 3}, false);
  std::vector<int> same(24, 3);
  same[0] = same[8] = same[16] = 52;
  check("dense heads on one XCD", 52, same, false);
  std::vector<int> two(16, 9);
  two[13] = 90;   // the first group is alike, the second is not
  check("one dense head of sixteen", 141, two, false);
  check("one head with entries", 5, {0, 0, 0, 0, 0, 0, 0, 5}, false);
  for (int i = 0; i < 4; ++i) {   // rules of the launchers: heads of at most 8 MiB, a multiple of 8
    const int D = i & 1 ? 128 : 64, block = i & 2 ? 128 : 64;
    const int fits = (int)(ut::kXcdHeadBytes / (4 * D));
    const struct { int N, H; bool heads; } rules[] = {
        {fits, 24, true}, {fits + 1, 24, false}, {1, 8, true}, {1, 12, false}, {fits, 20, false}};
    for (const auto& r : rules) {
      const ut::AttnShape sh{1, r.N, r.H, D, block, (r.N + block - 1) / block, 1.f};
      // dQ from the stored tiles: also a head's tiles in 8 MiB, but at 128 / 128
      const int64_t fit = ut::kXcdTileBytes / (2 * block * block) * r.H;
      const bool always = D == 128 && block == 128;
      const bool ok = ut::heads_by_xcd(sh) == r.heads && ut::stored_dq_by_head(sh, fit) == r.heads &&
                      ut::stored_dq_by_head(sh, fit + r.H) == (r.heads && always);
      std::printf("rules: %d tokens, %d heads of %d, block %d  %s\n", r.N, r.H, D, block, ok ? "ok" : "FAIL");
      if (!ok) ++failures;
    }
  }
  std::printf("%d failure(s)\n", failures);
  return failures != 0;
}
