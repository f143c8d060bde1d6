// Prints blocks per workgroup and workspace bytes of the packed training mask
// (tv_plan.h, pack_plan) for each "B A S Hq Hkv" on stdin.
#include <cstdio>
#include "tv_plan.h"

int main() {
  int B, A, S, Hq, Hkv;
  while (std::scanf("%d %d %d %d %d", &B, &A, &S, &Hq, &Hkv) == 5) {
    const tv::PackPlan p = tv::pack_plan(B, A, S, Hq, Hkv);
    std::printf("%d %d %zu\n", p.nb, p.packs, p.ws_bytes);
  }
  return 0;
}
