// Host-side half of the C-ABI front end: argument validation, the attention work list, the
// key-slice suggestion, workspace layouts and the bookkeeping of the pinned staging slots.
// Nothing here calls HIP, so the file also builds with a plain host compiler and its
// sanitizers (tests do that).
#pragma once
#include <stddef.h>
#include <stdint.h>

#include <vector>

#include "mc.h"
#include "mc_types.h"

namespace mc {
namespace host {

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
inline bool aligned4(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 3u) == 0; }

mc_status check_params(const mc_attn_params* p);

// softmax scale (0 selects 1 / sqrt(head_dim)) times log2(e): the kernels form probabilities with exp2
float attn_scale_log2e(const mc_attn_params* p);

// upper bound on work items: per request and KV head, ceil(C_r * G / rows) <= C_r * G / rows + 1
size_t max_items(const mc_attn_params* p, int32_t batch, int64_t total_new_tokens, int32_t kv_splits = 1);

// bytes of work list + request table for that bound (what the *_workspace_bytes calls return)
size_t list_bytes(const mc_attn_params* p, int32_t batch, int64_t total_new_tokens, int32_t kv_splits = 1);

// Lengths of a batch: sign and range checks, sum of the new tokens, most pages any request
// with new tokens needs.
mc_status check_lens(const mc_attn_params* p, const int32_t* prefix_lens, const int32_t* new_lens, int32_t batch,
                     int64_t* total_new, int32_t* need_pages);

// Everything an attention launch checks besides the lengths.  split == false: the whole-row kernel
// writes out / lse.  split == true: the split kernel writes partials (out / lse unused).
mc_status check_attn_buffers(bool split, const void* q, const void* k_pool, const void* v_pool,
                             const int32_t* block_tables, int32_t batch, int32_t max_pages_per_req, int32_t need_pages,
                             const void* out, const float* lse, const float* o_parts, const float* lse_parts,
                             const void* workspace);

// sizes that must hold before a work list is built: row and item counts the kernels index with 32 bits
mc_status check_list_range(const mc_attn_params* p, int32_t batch, int64_t total_new, int32_t kv_splits);

// New tokens that the requests of a batch bring to a launch: all of them, or (a batch that is two launches) those of the requests
// with more than `above` and at most `most`, while q and out hold the rows of all.
struct NewLens {
  const int32_t* of;                  // [batch]
  int32_t above, most;
  NewLens(const int32_t* all) : NewLens(all, 0, INT32_MAX) {}
  NewLens(const int32_t* all, int32_t above, int32_t most) : of(all), above(above), most(most) {}
  int32_t operator[](int32_t r) const { return of[r] > above && of[r] <= most ? of[r] : 0; }
};

// Work list of an attention launch: one item per (request, KV head, tile of stacked rows) and, for
// split launches (kv_splits >= 1), per key slice - most keys first, dealt round-robin so that
// consecutive workgroup ids (which land on different XCDs) take different (request, KV head)
// streams and each XCD's L2 keeps one stream hot.  Lengths have been validated by the caller.
void build_work_list(const mc_attn_params* p, const int32_t* prefix_lens, NewLens new_lens, int32_t batch,
                     int32_t kv_splits, std::vector<AttnReq>& reqs, std::vector<AttnItem>& items);

// number of whole-row work items of a batch (the size of the list build_work_list makes for kv_splits == 0)
int64_t count_items(const mc_attn_params* p, const int32_t* new_lens, int32_t batch);

// Every request's stacked rows of a KV head fit one row tile; and then, whether the K and V rows the requests read outgrow
// the last-level cache.
bool few_rows(const mc_attn_params* p, NewLens new_lens, int32_t batch, int64_t tile_rows);
bool reads_once(const mc_attn_params* p, const int32_t* prefix_lens, NewLens new_lens, int32_t batch, int64_t tile_rows);

// How a list of n_items workgroups is launched, kept in a plan: as row tiles of 256 rows (0), by workgroups of 128 rows, one
// per item or two, by workgroups of 64 rows, four per item, or by those of the narrow form, as many per item as it may have rows for, or one of the
// fewest rows (kListNarrowLeast: no item has more).  Marks that no caller's own zeroed or filled struct holds by accident: a
// list of longer row tiles launched one workgroup per item would leave rows out.
constexpr int32_t kListFew = 0x4d434631, kListFewOnce = 0x4d434632, kListHalves = 0x4d434633, kListNarrow = 0x4d434634,
                  kListNarrowLeast = 0x4d434635, kListPairs = 0x4d434636;
constexpr int32_t kListApart = 0x4d44;        // upper half of the mark of a list of two launches (ApartMark)
// (items of a plan that is launched narrow or by pairs: their workgroups have to be counted with 32 bits)
constexpr int32_t kMostNarrowItems = INT32_MAX / (kAttnTileRows / kAttnLeastRows);
int32_t list_form(const mc_attn_params* p, const int32_t* prefix_lens, const int32_t* new_lens, int32_t batch,
                  int32_t kv_splits, int64_t n_items);
// the same where the batch's whole rows have been planned (null: there is no plan, or the list is of key slices)
struct ClassPlan;
int32_t planned_list_form(const mc_attn_params* p, const int32_t* prefix_lens, const int32_t* new_lens, int32_t batch,
                          const ClassPlan* plan, int64_t n_items);

// Workgroups that take a row tile of the narrow form, each a share of its columns, where there are `row_tiles` (x pieces) of them.
int32_t narrow_shares(const mc_attn_params* p, int64_t row_tiles);

// A plan handed back by the caller: made for these params, of the wanted form, not empty.
mc_status check_plan(const mc_attn_params* p, const mc_attn_plan* plan, bool want_split);

// the body of mc_prefill_attn_plan and of mc_prefill_attn_suggest_kv_splits
mc_status plan_items(const mc_attn_params* p, const int32_t* prefix_lens, const int32_t* new_lens, int32_t batch,
                     int32_t kv_splits, int32_t* items, int64_t capacity, int64_t* n_items);
int32_t suggest_kv_splits(const mc_attn_params* p, const int32_t* prefix_lens, const int32_t* new_lens,
                          int32_t batch);

// What a one-shot attention call of a small batch launches: classes of row tiles (mc_types.h), no list in device memory.
// Requests in order of falling prefix (their cheapest row tile), row tiles from the last one down, so that what starts
// last is short.  With max_part_rows > 0 row tiles may be cut along the keys into pieces whose partial results take at
// most that many rows: the cut with the least estimated time is taken, which may be none.
// false: more requests with new tokens than a launch has classes for.
struct ClassPlan {
  AttnClasses classes;
  // Workgroups of the narrow form, if that is sooner (0: it is not); `narrow` are its classes, whole rows or cut into up to
  // narrow_pieces pieces, and the launch takes them instead.  Their partial results take no more room than those of `classes`
  // or, with `keep_room`, than max_part_rows.
  int32_t narrow_wgs, narrow_pieces;
  AttnClasses narrow;
  int32_t n_wgs;          // workgroups of the attention launch
  int32_t most_pieces;    // 1: nothing is cut, no partial results, no merge
  int64_t part_rows;      // rows of partial results
  double ends;            // us, by the estimate; 0: no other form was weighed
};
bool plan_classes(const mc_attn_params* p, const int32_t* prefix_lens, NewLens new_lens, int32_t batch,
                  int64_t max_part_rows, ClassPlan* plan, bool keep_room = false);

// Whole rows as two launches: the requests of few rows by the narrow form, then the others by a form of theirs.  false: one
// launch (`one`, whole rows) is as soon.  A prepared list holds the items of the first launch, then those of the second
// (apart_list, which returns the mark of such a list); calls without room for partial results launch the same two by classes, so
// that both compute the same bits.
struct ApartPlan {
  int32_t line;           // most new tokens of a request of the first launch
  ClassPlan few, many;
};
bool plan_apart(const mc_attn_params* p, const int32_t* prefix_lens, const int32_t* new_lens, int32_t batch, const ClassPlan& one,
                ApartPlan* apart);
int32_t apart_list(const mc_attn_params* p, const int32_t* prefix_lens, const int32_t* new_lens, const ApartPlan& apart,
                   int32_t batch, std::vector<AttnItem>& items);
struct ApartMark {
  int32_t n_few, shares;                        // items of the first launch, workgroups a row tile
  bool least;                                   // 16-row workgroups there
  int32_t form;                                 // of the second
  static constexpr int32_t kForms[5] = {0, kListFew, kListFewOnce, kListHalves, kListPairs};
  int32_t packed() const {
    int32_t at = 0;
    while (kForms[at] != form) ++at;
    return kListApart << 16 | at << 13 | (int32_t)least << 12 | (shares >> 1) << 10 | n_few;
  }
  // false: another mark, or one that does not fit a list of n_items
  bool unpack(int32_t mark, int32_t n_items) {
    const int32_t at = mark >> 13 & 7, share = mark >> 10 & 3;
    if (mark >> 16 != kListApart || at >= 5 || share == 3) return false;
    n_few = mark & 1023;
    shares = share == 0 ? 1 : 2 * share;
    least = (mark >> 12 & 1) != 0;
    form = kForms[at];
    return n_few > 0 && n_few < n_items;
  }
};

// Workspace of the automatic form: [work list + request table | o_parts | lse_parts], each part
// starting at a multiple of 256 bytes.  The partial results have room for kv_splits parts of every row (kv_splits > 1)
// or for what the class plan cuts (kv_splits == 1: by whole rows there is nothing to gain from uniform slices, but a
// launch of few workgroups is cut all the same); without either the workspace is the minimal one.
struct AutoLayout {
  int32_t kv_splits;
  size_t list_bytes, o_off, lse_off, total;
  bool room;              // the bytes that are available are enough for all of it
  bool by_classes;        // plan says what to launch (without room: whole rows); false: uniform slices or whole rows from a list
  ClassPlan plan;
};
bool auto_layout(const mc_attn_params* p, const int32_t* prefix_lens, const int32_t* new_lens, int32_t batch,
                 AutoLayout* lay, size_t available = SIZE_MAX);

// Whether the prefix keys of a batch are made by one workgroup per request in one launch: most blocks and most tokens of
// any request.
bool hash_in_one_launch(int64_t max_blocks, int64_t max_tokens);

// arguments of a page copy (pack / unpack and their relatives): a, b source pair, c, d destination pair
mc_status check_copy(const void* a, const void* b, int64_t num_pages, int64_t page_bytes, const int32_t* ids,
                     int64_t n, const void* c, const void* d);

// Whether a kernel may read and write `bytes` of pinned host memory at `at` itself: all of them lie in the allocation of `size`
// bytes from `start`, and its flags are among those of plain pinned memory (portable, mapped, NUMA-local, coherent).  Memory that is
// not coherent has a registered twin whose flag is another (coarse-grained: 0x8, also read-only); write-combined and I/O memory
// share a flag.  What is not named here goes by the copy engine.
constexpr uint32_t kPlainHostFlags = 0x60000003;
bool kernel_may_reach(uint32_t flags, uintptr_t at, uintptr_t start, size_t size, size_t bytes);

// Bookkeeping of the pinned host slots that work lists and tables are written to before their
// asynchronous upload.  A slot is FREE, HELD by a call that is filling it (between acquire and
// the event recorded behind its upload), or IN FLIGHT (its event decides when it is free again).
// A held slot is never handed out, whichever thread asks: the state is set under the owner's
// lock when the slot is picked, not when the upload has been enqueued.  The events and the
// memory themselves belong to the owner; this class only decides which slot a call gets.
class SlotRing {
 public:
  static constexpr int kMaxSlots = 256;
  enum State : int { kFree = 0, kHeld = 1, kInFlight = 2 };
  struct Pick {
    int slot;        // index, or -1: the ring is full of held slots or of other devices' slots
    bool is_new;     // the owner has to create the slot's event (and memory) first
    bool must_wait;  // every slot of the device is in flight and the ring is full: wait for this one's event
  };
  // `done(i)` tells whether the event of in-flight slot i has completed.  The returned slot is HELD.
  template <class Done>
  Pick pick(int dev, Done&& done) {
    const int n = n_;
    for (int k = 0; k < n; ++k) {
      const int i = (next_ + k) % n;
      if (dev_[i] != dev || state_[i] == kHeld) continue;
      if (state_[i] == kFree || done(i)) return take(i, false, false);
    }
    if (n < kMaxSlots) {
      dev_[n] = dev;
      ++n_;
      return take(n, true, false);
    }
    for (int k = 0; k < n; ++k) {
      const int i = (next_ + k) % n;
      if (dev_[i] == dev && state_[i] == kInFlight) return take(i, false, true);
    }
    return Pick{-1, false, false};
  }
  // the upload from the slot has been enqueued and its event recorded
  void in_flight(int slot) { state_[slot] = kInFlight; }
  // the call gave up before anything was enqueued from the slot (or its event could not be recorded
  // and the owner has waited for the stream instead)
  void abandon(int slot) { state_[slot] = kFree; }
  // a new slot whose event could not be created is taken out again (it is the last one)
  void drop_new(int slot) {
    if (slot == n_ - 1) --n_;
    else state_[slot] = kFree;
  }
  int size() const { return n_; }
  State state(int slot) const { return (State)state_[slot]; }
  int device(int slot) const { return dev_[slot]; }

 private:
  Pick take(int i, bool is_new, bool must_wait) {
    state_[i] = kHeld;
    next_ = (i + 1) % n_;
    return Pick{i, is_new, must_wait};
  }
  int n_ = 0, next_ = 0;
  int dev_[kMaxSlots] = {};
  int state_[kMaxSlots] = {};
};

}  // namespace host
}  // namespace mc
