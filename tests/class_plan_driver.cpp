// Prints the class plan of each batch read from stdin, one line per plan (tests/test_class_plan.py checks them).
// input:  Hq Hkv D dtype max_part_rows batch P... C...
// output: n n_wgs most_pieces part_rows tile_rows [first req q_off prefix chunk tile_lo tile_hi pieces part_base]...
//         and the rows of a workgroup of the launch (of its narrow form, if it takes that) and of the prepared list of the batch
#include <cstdio>
#include <vector>

#include "host_plan.h"

int main() {
  int Hq, Hkv, D, dtype, batch;
  long long max_part_rows;
  while (std::scanf("%d %d %d %d %lld %d", &Hq, &Hkv, &D, &dtype, &max_part_rows, &batch) == 6) {
    std::vector<int32_t> P(batch), C(batch);
    for (auto& x : P)
      if (std::scanf("%d", &x) != 1) return 1;
    for (auto& x : C)
      if (std::scanf("%d", &x) != 1) return 1;
    const mc_attn_params p{Hq, Hkv, D, 16, 1 << 20, dtype, 0.f};
    mc::host::ClassPlan plan;
    if (!mc::host::plan_classes(&p, P.data(), C.data(), batch, max_part_rows, &plan)) {
      std::printf("none\n");
      continue;
    }
    std::printf("%d %d %d %lld %d", plan.classes.n, plan.n_wgs, plan.most_pieces, (long long)plan.part_rows, plan.classes.rows);
    for (int i = 0; i < plan.classes.n; ++i) {
      const mc::AttnClass& k = plan.classes.c[i];
      std::printf(" %d %d %d %d %d %d %d %d %d", plan.classes.first[i], k.req, k.q_off, k.prefix, k.chunk, k.tile_lo, k.tile_hi,
                  k.pieces, k.part_base);
    }
    const int32_t form = mc::host::list_form(&p, P.data(), C.data(), batch, 0, mc::host::count_items(&p, C.data(), batch));
    // as launch_planned_attn and launch_attn read it
    const int narrow = dtype == MC_DTYPE_F32 ? mc::kAttnLeastRows : mc::kAttnNarrowRows;
    const int list = form == 0 ? mc::kAttnTileRows : form == mc::host::kListNarrowLeast ? mc::kAttnLeastRows
                   : form == mc::host::kListNarrow ? narrow
                   : form == mc::host::kListPairs ? mc::kAttnPairRows : mc::kAttnFewRows;
    std::printf(" %d %d\n", plan.narrow_wgs > 0 ? plan.narrow.rows : plan.classes.rows, list);
  }
  return 0;
}
