// Plans each batch read from stdin as a call without room for partial results does (plan_classes, then plan_apart); one line a
// batch: "none" (more requests than classes), "one" or "two" launches.
// input:  Hq Hkv D dtype batch P... C...
#include <cstdio>
#include <vector>

#include "host_plan.h"

int main() {
  int Hq, Hkv, D, dtype, batch;
  while (std::scanf("%d %d %d %d %d", &Hq, &Hkv, &D, &dtype, &batch) == 5) {
    std::vector<int32_t> P(batch), C(batch);
    for (auto& x : P)
      if (std::scanf("%d", &x) != 1) return 1;
    for (auto& x : C)
      if (std::scanf("%d", &x) != 1) return 1;
    const mc_attn_params p{Hq, Hkv, D, 16, 1 << 20, dtype, 0.f};
    mc::host::ClassPlan one;
    mc::host::ApartPlan apart;
    if (!mc::host::plan_classes(&p, P.data(), C.data(), batch, 0, &one)) {
      std::puts("none");
      continue;
    }
    std::puts(mc::host::plan_apart(&p, P.data(), C.data(), batch, one, &apart) ? "two" : "one");
  }
  return 0;
}
