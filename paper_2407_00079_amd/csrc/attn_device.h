// Device-side pieces shared by the attention kernels: vector types, tile geometry in LDS, the
// direct global -> LDS copy and the exchange between the two halves of a wave.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mc_types.h"

namespace mc {
namespace {

typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4;
typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

#define MC_LDS __attribute__((address_space(3)))

constexpr int kWaves = 8;              // waves of a workgroup: two per SIMD, 32 stacked rows each
static_assert(kWaves * 32 == kAttnTileRows, "the host cuts the work list into tiles of kAttnTileRows rows");
constexpr int kTileKeys = kAttnTileKeys;   // keys per LDS tile = 4 pages of 16
constexpr int kPageTokens = 16;
constexpr int kRowBytes = 256;         // one K or V row: 128 bf16 or 64 f32
constexpr int kPageHeadBytes = kPageTokens * kRowBytes;   // 4 KiB, contiguous in the pool
constexpr int kKTileBytes = kTileKeys * kRowBytes;        // 16 KiB; rows dense, granules swizzled
constexpr int kVTileBytes = kTileKeys * kRowBytes;
constexpr int kBuffers = 3;
constexpr int kDeepBuffers = 4;        // 128 KiB of 256-byte rows, of 160 KiB a compute unit has
// LDS: the K tiles of the three buffers, then the V tiles.  Every tile starts at a multiple of
// 16 KiB, so the XOR constants of the swizzle (< 256) never reach a tile base, and the offset of
// any fragment from its lane's base register stays below the 64 KiB a ds_read immediate can hold.
constexpr int kVBase = kBuffers * kKTileBytes;
constexpr float kRescaleSlack = 8.0f;  // log2 units the running max may lag behind
// stands in for a reference of -inf when probabilities are formed: masked scores (-inf) then give
// exp2(-inf) = 0 instead of exp2(-inf + inf) = NaN; a row with a finite score has a finite reference
constexpr float kNoKeyYet = -1e30f;

// Which waves do what.  Full tiles (256 rows): all eight compute, the first of each SIMD copies tiles besides (it wins the
// issue arbitration and would idle at the tile barrier).  Few rows (128): the first of each SIMD computes, the second only
// copies; a copy instruction holds its wave for about 130 cycles, which a lone computing wave has no one to hide behind
// (16 tokens at 128k, 64/8 heads: 115 us a call with four waves that do both, 97 with four and four).
// Full tiles / few rows, one call, bf16 head_dim 128, 64/8 heads unless said: P 131056, C 16 111 / 96 us; P 131056, C 1
// 101 / 86; P 1000, C 100 28 / 22; P 256, C 128 17 / 13; P 30000, C 300 245 / 275; head_dim 64, P 131056, C 16 69 / 60;
// fp32, 4/1 heads, P 256, C 128 24 / 17, P 6955, C 200 80 / 46.
// Pair rows (64): as few rows, but the four that compute are two pairs, one for the first 32 keys of every tile and one for the
// others; their results meet in LDS at the end.
enum Rows { kFullRows = 0, kFewRows = 1, kPairRows = 2 };
constexpr int kFetchWaves = 4;
template <Rows R>
constexpr int kTileRowsOf = R == kPairRows ? kAttnPairRows : R == kFewRows ? kAttnFewRows : kAttnTileRows;
template <Rows R>
__device__ __forceinline__ bool wave_copies(int wave) { return R != kFullRows ? wave >= kFetchWaves : wave < kFetchWaves; }
template <Rows R>
__device__ __forceinline__ bool wave_computes(int wave) { return R == kFullRows || wave < kFetchWaves; }

// How a launch describes its work: whole rows or uniform key slices from a list in device memory, or classes from the
// kernel argument.
enum Form { kWhole = 0, kSlices = 1, kClasses = 2 };

// One workgroup's work, whatever described it.  The key tiles are cut into `pieces` (classes) or the request's tiles
// into a.kv_splits slices of which this is number `piece` (slices); `part_row` + stacked row (classes) or + output row
// (slices) is where a partial result goes.
struct Work {
  int32_t req, kv_head, row0, q_off, prefix, chunk;
  int32_t piece, pieces;
  int64_t part_row;
  bool once;                             // K and V are streamed (AttnClasses::once)
};

// list launches; workgroups n_items .. take the second halves of the items' row tiles (few rows).  Pair rows: the quarters of eight
// items together, in the order of the list and each on its item's XCD (the last n_items % 8 items: one quarter after another).
template <Rows R, typename Args>
__device__ __forceinline__ Work work_of(const Args& a, int wg) {
  if constexpr (R == kPairRows) {
    constexpr int kParts = kAttnTileRows / kAttnPairRows;
    const int rest = a.n_items % kXcds, whole = (a.n_items - rest) * kParts, behind = wg - whole;
    const int part = behind < 0 ? wg / kXcds % kParts : behind / rest;
    const AttnItem item = a.items[behind < 0 ? wg / (kXcds * kParts) * kXcds + wg % kXcds : a.n_items - rest + behind % rest];
    const AttnReq rq = a.reqs[item.req];
    return Work{item.req, item.kv_head, item.row0 + part * kAttnPairRows, rq.q_off, rq.prefix, rq.chunk, 0, 1, 0, false};
  }
  const bool second = R == kFewRows && wg >= a.n_items;
  const AttnItem item = a.items[second ? wg - a.n_items : wg];
  const AttnReq rq = a.reqs[item.req];
  return Work{item.req, item.kv_head, item.row0 + (second ? kAttnFewRows : 0), rq.q_off, rq.prefix, rq.chunk, item.slice, 1,
              (int64_t)item.slice * a.rows_total, a.once != 0};
}

// the class of workgroup (or merge block) wg: the last one whose first is not past it
__device__ __forceinline__ int class_of(const AttnClasses& t, int wg) {
  const int lane = threadIdx.x & 63;
  const int first = t.first[lane];
  return __popcll(__builtin_amdgcn_ballot_w64(lane < t.n && first <= wg)) - 1;
}
__device__ __forceinline__ int class_rows(const AttnClass& k, int G, int tile_rows) {
  const int all = k.chunk * G, hi = (k.tile_hi + 1) * tile_rows;
  return (all < hi ? all : hi) - k.tile_lo * tile_rows;
}
template <int TILE_ROWS>
__device__ __forceinline__ Work work_of(const AttnClasses& t, int wg, int Hkv, int G) {
  const int at = class_of(t, wg);
  const AttnClass k = t.c[at];
  const int local = wg - t.first[at];
  const int head = local % Hkv, rest = local / Hkv;
  const int piece = rest % k.pieces, row0 = (k.tile_hi - rest / k.pieces) * TILE_ROWS;
  const int64_t part = (int64_t)k.part_base + (int64_t)(piece * Hkv + head) * class_rows(k, G, TILE_ROWS) - k.tile_lo * TILE_ROWS;
  return Work{k.req, head, row0, k.q_off, k.prefix, k.chunk, piece, k.pieces, part, t.once != 0};
}
// key tiles [lo, hi) of the n a row tile sees that piece `piece` of `pieces` covers
__device__ __forceinline__ void piece_tiles(int n, int piece, int pieces, int* lo, int* hi) {
  const int each = n / pieces, more = n - each * pieces;
  *lo = piece * each + (piece < more ? piece : more);
  *hi = *lo + each + (piece < more ? 1 : 0);
}

// Combine a value with the one held by lane ^ 32.  v_permlane32_swap exchanges the upper
// half of its first register with the lower half of its second, so after it every lane
// holds its own value in one register and its partner's in the other; max and sum do not
// care which is which.  Written as asm with two distinct read-write registers (the builtin
// called with one value for both operands gets its two results merged by the optimiser);
// the s_nop covers the VALU-write -> permlane read hazard the compiler cannot see.
__device__ __forceinline__ void swap_halves(float& a, float& b) {
  asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1\n\ts_nop 1" : "+v"(a), "+v"(b));
}
__device__ __forceinline__ float max_with_other_half(float x) {
  float a = x, b = x;
  swap_halves(a, b);
  return fmaxf(a, b);
}
__device__ __forceinline__ float sum_with_other_half(float x) {
  float a = x, b = x;
  swap_halves(a, b);
  return a + b;
}

// Direct global -> LDS copy of 16 bytes per lane: lane i's bytes land at lds_base + 16*i
// (lds_base wave-uniform, it travels in M0).  Written as asm so that the compiler does not
// know LDS is being written behind its back: it would otherwise make the first LDS read
// after the copy wait for the copy (vmcnt), which is exactly what the tile pipeline avoids.
// Ordering is the kernel's own business: s_waitcnt vmcnt(0) + barrier before a tile is read.
// (M0 is a register the compiler reserves for itself; it sets it right before each of its own
// uses and has none in this kernel, so naming it as clobbered is all that is needed - the
// diagnostic about reserved registers in a clobber list is expected here.)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void dma16(const char* sbase, uint32_t voff, uint32_t lds_base) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %0"
               :: "s"(sbase), "v"(voff), "s"(lds_base) : "m0", "memory");
}
__device__ __forceinline__ void dma16(const char* vaddr, uint32_t lds_base) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off"
               :: "v"(vaddr), "s"(lds_base) : "m0", "memory");
}
// The chunks of a page (1 KiB each, contiguous in the pool and in LDS): the immediate offset of the instruction advances
// the global and the LDS address alike, so one base and one M0 serve all of them.  ONCE: the bytes are not read again soon.
#define MC_COPY_PAGE_4(HINT)                                                                                              \
  asm volatile("s_mov_b32 m0, %5\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %0" HINT "\n\t"                              \
               "global_load_lds_dwordx4 %2, %0 offset:1024" HINT "\n\tglobal_load_lds_dwordx4 %3, %0 offset:2048" HINT    \
               "\n\tglobal_load_lds_dwordx4 %4, %0 offset:3072" HINT                                                      \
               :: "s"(sbase), "v"(voff[0]), "v"(voff[1]), "v"(voff[2]), "v"(voff[3]), "s"(lds_base) : "m0", "memory")
#define MC_COPY_PAGE_2(HINT)                                                                                              \
  asm volatile("s_mov_b32 m0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %0" HINT "\n\t"                              \
               "global_load_lds_dwordx4 %2, %0 offset:1024" HINT                                                          \
               :: "s"(sbase), "v"(voff[0]), "v"(voff[1]), "s"(lds_base) : "m0", "memory")
template <bool ONCE, int CHUNKS>
__device__ __forceinline__ void dma16_page(const char* sbase, const uint32_t (&voff)[CHUNKS], uint32_t lds_base) {
  static_assert(CHUNKS == 2 || CHUNKS == 4, "a page is 2 or 4 KiB");
  if constexpr (CHUNKS == 4) {
    if constexpr (ONCE) MC_COPY_PAGE_4(" nt");
    else MC_COPY_PAGE_4("");
  } else {
    if constexpr (ONCE) MC_COPY_PAGE_2(" nt");
    else MC_COPY_PAGE_2("");
  }
}
#undef MC_COPY_PAGE_4
#undef MC_COPY_PAGE_2
#pragma clang diagnostic pop

}  // namespace
}  // namespace mc
