// Host time of planning a one-shot attention call of dozens of requests, against building the list of the same batch
// (tests/test_class_plan.py): prints "plan_us list_us" per batch read from stdin.  WHOLE_ROWS: of planning one without room for
// partial results, two launches included.
// input:  Hq Hkv D dtype batch P... C...
#include <chrono>
#include <cstdio>
#include <vector>

#include "host_plan.h"

template <class F>
static double least_us(F f) {
  double least = 1e9;
  for (int k = 0; k < 200; ++k) {
    const auto t0 = std::chrono::steady_clock::now();
    f();
    const double us = std::chrono::duration<double, std::micro>(std::chrono::steady_clock::now() - t0).count();
    least = us < least ? us : least;
  }
  return least;
}

int main() {
  int Hq, Hkv, D, dtype, batch;
  while (std::scanf("%d %d %d %d %d", &Hq, &Hkv, &D, &dtype, &batch) == 5) {
    std::vector<int32_t> P(batch), C(batch);
    for (auto& x : P)
      if (std::scanf("%d", &x) != 1) return 1;
    for (auto& x : C)
      if (std::scanf("%d", &x) != 1) return 1;
    const mc_attn_params p{Hq, Hkv, D, 16, 1 << 20, dtype, 0.f};
    std::vector<mc::AttnReq> reqs;
    std::vector<mc::AttnItem> items;
#ifdef WHOLE_ROWS
    mc::host::ClassPlan one;
    mc::host::ApartPlan apart;
    const double plan = least_us([&] {
      if (mc::host::plan_classes(&p, P.data(), C.data(), batch, 0, &one)) mc::host::plan_apart(&p, P.data(), C.data(), batch, one, &apart);
    });
#else
    mc::host::AutoLayout lay;
    const double plan = least_us([&] { mc::host::auto_layout(&p, P.data(), C.data(), batch, &lay); });
#endif
    const double list = least_us([&] { mc::host::build_work_list(&p, P.data(), C.data(), batch, 0, reqs, items); });
    std::printf("%.2f %.2f\n", plan, list);
  }
  return 0;
}
