// Plain data shared by the host-side planning code and the kernels: no HIP types here, so that the
// planning code also builds with an ordinary host compiler (and its sanitizers).
#pragma once
#include <stdint.h>

namespace mc {

// One unit of attention work: a tile of stacked query rows of one (request, KV head).
// Stacked row index = token_in_chunk * G + head_in_group, so one K/V tile in LDS
// feeds all G query heads of the group.
struct AttnItem {
  int32_t req;
  int32_t kv_head;
  int32_t row0;   // first stacked row of the tile
  int32_t slice;  // key slice of the request this item covers (split launches only, else 0)
};

struct AttnReq {
  int32_t q_off;   // index of the request's first new token in q / out
  int32_t prefix;  // P_r
  int32_t chunk;   // C_r
  int32_t pages;   // ceil((P_r + C_r) / S): entries of the block-table row that may be read
};

// A run of row tiles of one request that are all cut into the same number of pieces along the keys: what an attention
// launch of a small batch is described with.  A launch has at most a few dozen of them, so they travel as a kernel
// argument (no list in device memory, no upload); every workgroup finds its class and its place in it by arithmetic.
// What that is worth: the upload of a list cost a copy kernel of 4 us and gaps of 5-6 us up to 16 KiB, gaps of 20-30 us
// above (copy engine); P 8189, C 4099 (1032 workgroups, head_dim 64) went from 699 to 688 us with it gone.
// Workgroups of a class, from its first one on: KV heads fastest (consecutive workgroups land on different XCDs, so an
// XCD keeps the K/V stream of one head), then pieces, then row tiles from tile_hi down to tile_lo (most keys first).
// pieces == 1: the tile's output is final.  pieces > 1: piece i covers tiles [i n / pieces, (i + 1) n / pieces) of the n
// key tiles the row tile sees (the first n % pieces pieces one more than the rest) and writes row x of head g to row
// part_base + (i Hkv + g) rows + x of the partial results, rows = the class's stacked rows per head.
struct AttnClass {
  int32_t req, q_off, prefix, chunk;
  int32_t tile_lo, tile_hi;
  int32_t pieces;
  int32_t part_base;
};
constexpr int kMaxAttnClasses = 64;          // one lane of a wave each when a workgroup looks for its class
struct AttnClasses {
  int32_t n;
  int32_t rows;                              // stacked rows of a row tile: kAttnTileRows, kAttnFewRows, kAttnNarrowRows or kAttnLeastRows
  int32_t once;                              // K and V are streamed: one row tile per head, more bytes than the caches hold
  int32_t first[kMaxAttnClasses];            // first workgroup of each class (of the attention launch or of the merge)
  AttnClass c[kMaxAttnClasses];
};

// Small host tables travel in the kernel argument instead of being uploaded first: the upload cost the host 7-8 us a call
// (staging slot, copy, event; small calls are bound by the host) and the GPU a copy kernel of 2-4 us and its gaps.  64
// entries, one lane of a wave each, are 1 KiB of argument; longer tables are still uploaded.  One pass before / after, us:
// append + attention of the tiny fp32 request 33.4 / 26.7, of 16 tokens at 128k 117 / 111; keys + match of one prompt of
// 6955 tokens 35.6 / 25.5, of 64 prompts of 128k tokens 72.2 / 59.8.
constexpr int kMaxArgEntries = 64;
struct AttnReqTable {
  AttnReq r[kMaxArgEntries];
};
// two offset tables of at most kMaxArgEntries + 1 entries each
struct OffsetTables {
  int64_t a[kMaxArgEntries + 1], b[kMaxArgEntries + 1];
};

// most blocks of a request whose keys one workgroup makes in one launch (its digests go through LDS)
constexpr int kShortHashBlocks = 32;

// rows of stacked queries one attention workgroup covers (8 waves of 32 rows, both dtypes)
constexpr int kAttnTileRows = 256;
// ... and of the form for launches whose row tiles are few or short: 4 waves compute (one per SIMD), 4 copy tiles
constexpr int kAttnFewRows = 128;
// ... and of the one between that and the narrow form: the waves that compute are two pairs, each for every other 32 keys (bf16)
constexpr int kAttnPairRows = 64;
// ... and of the narrow form, whose waves share out keys instead of rows (attn_narrow.hip): bf16, or fp32 and bf16 where no
// request has more rows
constexpr int kAttnNarrowRows = 32, kAttnLeastRows = 16;
// keys of one LDS tile; key slices of the split form are whole tiles
constexpr int kAttnTileKeys = 64;
// 16-byte vectors of a page one copy workgroup moves (512 threads, one vector each)
constexpr int kKvCopySliceVecs = 512;
// bytes of a page that a workgroup of a small load or store against host memory moves at a time, and the most such slices of K
// of a call that goes that way: 2 MiB (kv_host_kernel in kv_copy.hip)
constexpr int kHostSliceBytes = 4096;
constexpr int64_t kMostHostSlices = 512;
// the work list is kept in this many lists, one per XCD of the chip
constexpr int kXcds = 8;

}  // namespace mc
