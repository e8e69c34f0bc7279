// Internal declarations shared by the C-ABI front end and the gfx950 kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mc.h"
#include "mc_types.h"

namespace mc {

struct AttnArgs {
  const void* q;
  const void* k_pool;
  const void* v_pool;
  const int32_t* block_tables;
  void* out;
  float* lse;
  const AttnItem* items;
  const AttnReq* reqs;
  int32_t Hq, Hkv, G, max_pages;
  int32_t head_dim;   // bf16: 128 or 64; fp32: 64
  float scale_log2e;  // softmax scale * log2(e): scores go through exp2
  int32_t n_items;
  int32_t few_rows;    // list launches: 128-row workgroups, one per item (no item has more rows) or two (halves)
  int32_t halves;
  int32_t pair_rows;   // list launches (bf16): 64-row workgroups, four per item
  int32_t once;        // list launches: as AttnClasses::once
  // split launches (kv_splits > 0): partial results go to o_parts [kv_splits, rows_total, D] fp32 and
  // lse_parts [kv_splits, rows_total] instead of out / lse
  int32_t kv_splits;
  int64_t rows_total;  // total_new_tokens * Hq
  float* o_parts;
  float* lse_parts;
};

// enqueue the attention kernel over args.n_items work items
hipError_t launch_attn(int dtype, const AttnArgs& args, hipStream_t stream);

// the bf16 instantiation (attn_prefill_bf16.hip), reached through launch_attn
hipError_t launch_attn_bf16(const AttnArgs& args, hipStream_t stream);

// the same over args.n_items workgroups described by classes (args.items, reqs and kv_splits unused)
hipError_t launch_attn_classes(int dtype, const AttnArgs& args, const AttnClasses& t, hipStream_t stream);
hipError_t launch_attn_bf16_classes(const AttnArgs& args, const AttnClasses& t, hipStream_t stream);

// the narrow form: args.n_items workgroups described by classes of its row tiles, or (t null) the row tiles of the list's
// args.n_items items, whole, `parts` row tiles an item; rows of a workgroup: kAttnNarrowRows (bf16) or kAttnLeastRows;
// `shares` workgroups a row tile, each for as many of the output's columns: 1, 2 or 4
hipError_t launch_attn_narrow(int dtype, const AttnArgs& args, int rows, int parts, int shares, const AttnClasses* t,
                              hipStream_t stream);

// enqueue the merge of the classes that were cut into pieces (nothing if none was)
hipError_t launch_attn_merge_classes(int dtype, int head_dim, const float* o_parts, const float* lse_parts,
                                     const AttnClasses& all, int Hq, int Hkv, void* out, float* lse, hipStream_t stream);

// enqueue the merge of kv_splits partial results over `rows` rows into out (dtype) and lse (or null)
hipError_t launch_attn_merge(int dtype, int head_dim, const float* o_parts, const float* lse_parts, int kv_splits, int64_t rows,
                             void* out, float* lse, hipStream_t stream);

// enqueue gather (pack) or scatter (unpack) of n pages of page_bytes for K and V; `order` (or null)
// lists the positions of page_ids in the order the workgroups should take them
hipError_t launch_kv_copy(bool pack, const void* k_src, const void* v_src, void* k_dst, void* v_dst,
                          const int32_t* page_ids, const int32_t* order, int64_t n, int64_t page_bytes,
                          hipStream_t stream);

// enqueue a layer's load from (or store to) host memory that the device sees at k_host, v_host: host and stage hold the n pages
// in list order.  For small n (2 n ceil(page_bytes / kHostSliceBytes) has to fit 32 bits).
hipError_t launch_kv_host(bool load, void* k_host, void* v_host, void* k_stage, void* v_stage, void* k_pool, void* v_pool,
                          const int32_t* page_ids, int64_t n, int64_t page_bytes, hipStream_t stream);

// enqueue the computation of order[r] = position of the r-th smallest page id (stable)
hipError_t launch_kv_page_order(const int32_t* page_ids, int64_t n, int32_t* order, hipStream_t stream);

// enqueue the count of ids outside [0, num_pages) into report[0] and the first such position (n if none) into report[1]
hipError_t launch_kv_check_page_ids(const int32_t* page_ids, int64_t n, int64_t num_pages, int32_t* report,
                                    hipStream_t stream);

// enqueue the scatter of total_new tokens' K/V rows (row_bytes = 256 or 128 per KV head) into their page slots; the
// request table is in device memory (reqs) or, for at most kMaxArgEntries requests, travels with the launch (arg)
hipError_t launch_kv_append(const void* k_new, const void* v_new, void* k_pool, void* v_pool,
                            const int32_t* block_tables, int32_t max_pages, const AttnReq* reqs, const AttnReqTable* arg,
                            int32_t batch, int64_t total_new, int32_t Hkv, int32_t row_bytes, hipStream_t stream);

// The offset tables of a prefix call: both in device memory or, if `arg` is set, both in it (at most kMaxArgEntries + 1
// entries each; they then travel with the launch).
struct PrefixTables {
  const int64_t *a, *b;
  const OffsetTables* arg;
};

// enqueue the kernels that turn tokens into keys (tables: token offsets, key offsets; max_blocks = most blocks of any
// request, total_blocks = all of them, in_one_launch: no request has more than kShortHashBlocks and it pays)
hipError_t launch_prefix_hash(const int32_t* tokens, const PrefixTables& tables, int batch, int block_tokens,
                              int64_t max_blocks, int64_t total_blocks, bool in_one_launch, uint64_t* keys,
                              hipStream_t stream);

// enqueue the prefix match over batch requests and n_inst instances (tables: key offsets, cache offsets; max_keys = most
// keys of any request)
hipError_t launch_prefix_match(const uint64_t* keys, const PrefixTables& tables, int batch, int64_t max_keys,
                               const uint64_t* cache_keys, int n_inst, int32_t* prefix_len, int32_t* best_len,
                               int32_t* best_inst, hipStream_t stream);

}  // namespace mc
