// Host check of the even split's work order (tv_plan.h): for "count slots nRB
// Hkv" on stdin, decodes every workgroup of the plan's grid for that many
// slots and verifies that the first `count` chunks of every (KV head, row
// block) are taken exactly once, and that a chunk's row blocks share an XCD.
#include <cstdio>
#include <vector>
#include "tv_plan.h"

int main() {
  int count, slots, nRB, Hkv, bad = 0, cases = 0;
  while (std::scanf("%d %d %d %d", &count, &slots, &nRB, &Hkv) == 4) {
    ++cases;
    const int grid = tv::kXcds * nRB * tv::cdiv((long long)slots * Hkv, tv::kXcds);
    std::vector<int> seen((size_t)count * nRB * Hkv, 0), xcd((size_t)count * Hkv, -1);
    bool ok = true;
    for (int bid = 0; bid < grid; ++bid) {
      tv::WorkItem it{};
      const int item = tv::even_item(bid, count, nRB, Hkv, it);
      if (item < 0) continue;
      if (item >= count || it.g < 0 || it.g >= Hkv || it.rb < 0 || it.rb >= nRB) {
        ok = false;
        break;
      }
      seen[(size_t)(item * Hkv + it.g) * nRB + it.rb]++;
      int& x = xcd[(size_t)item * Hkv + it.g];
      ok = ok && (x == -1 || x == bid % tv::kXcds);
      x = bid % tv::kXcds;
    }
    for (int v : seen) ok = ok && v == 1;
    if (!ok) std::printf("FAIL count=%d slots=%d nRB=%d Hkv=%d\n", count, slots, nRB, Hkv);
    bad += !ok;
  }
  std::printf("%d cases, %d failed\n", cases, bad);
  return bad ? 1 : 0;
}
