// Plans each batch read from stdin as a call without room for partial results does (plan_classes, then plan_apart); one line a
// batch: "none" (more requests than classes), "one" or "two" launches, the allocations on the host heap that both planning functions
// made, and of one launch the rows of its workgroups (0: narrow) and its estimated end in microseconds,
// and whether a list's form is the same from that plan as from the lengths.
// With an argument, of each batch of two launches only: "line | rows of a workgroup, then classes, of the first launch | the same
// of the second | the list's mark, then what it is read as | the list's items", numbers all.
// input:  Hq Hkv D dtype batch P... C...
#include <cstdio>
#include <cstdlib>
#include <new>
#include <vector>

#include "host_plan.h"

static long news = 0;
#ifdef COUNT_NEWS            // (MemorySanitizer has its own)
void* operator new(size_t bytes) {
  ++news;
  void* p = std::malloc(bytes);
  if (p == nullptr) throw std::bad_alloc();
  return p;
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }
#endif

static void print(const mc::AttnClasses& t) {
  std::printf(" | %d", t.rows);
  for (int i = 0; i < t.n; ++i)
    std::printf(" %d %d %d %d %d %d %d %d", t.first[i], t.c[i].req, t.c[i].q_off, t.c[i].prefix, t.c[i].chunk, t.c[i].tile_lo,
                t.c[i].tile_hi, t.c[i].pieces);
}

static void print_two(const mc_attn_params& p, const std::vector<int32_t>& P, const std::vector<int32_t>& C,
                      const mc::host::ApartPlan& apart) {
  std::printf("%d", apart.line);
  print(apart.few.narrow);
  print(apart.many.classes);
  std::vector<mc::AttnItem> items;
  const int32_t packed = mc::host::apart_list(&p, P.data(), C.data(), apart, (int32_t)P.size(), items);
  mc::host::ApartMark mark;
  const bool read = mark.unpack(packed, (int32_t)items.size()), small = mark.unpack(packed, mark.n_few);
  std::printf(" | %d %d %d %d %d %d %d", packed, read, small, mark.n_few, mark.shares, mark.least, mark.form);
  std::printf(" %d |", mc::host::narrow_shares(&p, apart.few.narrow_wgs));
  for (const mc::AttnItem& it : items) std::printf(" %d %d %d %d", it.req, it.kv_head, it.row0, it.slice);
  std::puts("");
}

int main(int argc, char**) {
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
    const long before = news;
    const bool planned = mc::host::plan_classes(&p, P.data(), C.data(), batch, 0, &one);
    const long by_classes = news - before;
    const bool two = planned && mc::host::plan_apart(&p, P.data(), C.data(), batch, one, &apart);
    if (argc > 1) {
      if (two) print_two(p, P, C, apart);
      else std::puts("");
      continue;
    }
    std::printf("%s %ld %ld", !planned ? "none" : two ? "two" : "one", by_classes, news - before - by_classes);
    std::printf(" %d %.9g", planned && one.narrow_wgs == 0 ? one.classes.rows : 0, planned ? one.ends : 0.0);
    const int64_t items = mc::host::count_items(&p, C.data(), batch);
    const bool form = mc::host::planned_list_form(&p, P.data(), C.data(), batch, planned ? &one : nullptr, items) ==
                      mc::host::list_form(&p, P.data(), C.data(), batch, 0, items);
    std::printf(" %d\n", form);
  }
  return 0;
}
