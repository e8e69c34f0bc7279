// bf16 instantiation of the prefix-reused, paged, chunked-prefill attention (paper Section 3,
// steps 1-2; the kernel design is ours) on 16x16x32 MFMA tiles.
//
// Why this tile shape.  The board holds its power limit by lowering the shader clock, and the
// energy of a bf16 MFMA per flop depends on its shape: a loop of v_mfma_f32_16x16x32_bf16 runs
// at ~2.0 GHz where the same flops as v_mfma_f32_32x32x16_bf16 run at ~1.75 GHz (a 16x16x32
// tile reads and writes a quarter of the accumulator registers per instruction and half per
// flop).  What a 16x16 tile would cost elsewhere - twice the operand fragments per flop - is
// avoided by giving every wave TWO row tiles: each K or V fragment read from LDS feeds two
// MFMAs, so the LDS traffic per flop is that of the 32x32 form.
//
// Shape of the computation (see attn_prefill.hip for what is common to both dtypes)
//   * A wave owns 32 stacked query rows as two row tiles of 16; lane l serves rows l % 16 of
//     both tiles and, of every 32-key block, the 8 keys 4 (l / 16) + {0..3} and 16 + 4 (l / 16)
//     + {0..3} - the rows of its lane group in the two 16x16 score tiles S^T = K Q^T.  The
//     probabilities of a lane are therefore already the B operand of O^T += V^T P^T (a 32-key
//     contraction in that key order); V^T fragments are fetched in the same order with two LDS
//     transpose reads.  Row maxima (diagonal tiles and the rare recompute path only) are in-lane
//     over 8 values plus an exchange between the 4 lane groups.
//   * Per 32-key block at head_dim 128: 16 score MFMAs (2 key tiles x 2 row tiles x 4 head_dim
//     steps of 32) and 16 P V MFMAs (8 head_dim tiles x 2 row tiles), 8 K fragments and 8 V
//     fragments from LDS; at head_dim 64 half of each (see Geo).
//   * K/V tiles, the page walk, the lazy softmax reference, the two-phase ring and the half-step
//     skew of the two waves of a SIMD are those of attn_prefill.hip; the swizzles differ (fragment
//     shapes differ), and so does what runs under which MFMAs.
//   * With two waves per SIMD an MFMA of this shape hides about two vector instructions of its
//     wave (one exp2 counts as two); a third costs more than its own issue time (stand-alone loop
//     of MFMA + n fma, two waves per SIMD: 33, 34, 34, 46 cycles per pair of MFMAs for n = 0..3).
//     The softmax is therefore kept to what it cannot do without - per score one fma and one exp2,
//     per pair one rounding to bf16 - and spread over BOTH phases: row tile 1 of block j under the
//     score MFMAs of block j+1, row tile 0 of block j+1 under the P V MFMAs of block j.  The row
//     sums of the rounded probabilities come from two more MFMAs per block (ones x P^T), and the
//     guard of the lazy reference is an OR over the packed probabilities (see kRefLift).
//   * Pair rows (64-row workgroups): for launches whose 128-row tiles leave compute units idle and whose 32-row ones would take
//     several rounds.  A tile is one block for each wave: 0.44-0.47 us (head_dim 64: 0.36), of which the copies hold the compute unit
//     for 0.29; 0.72 (0.55) with 128 rows.  The two pairs meet in LDS once, at the end.  Planned, us, before / so: 64/8 heads,
//     P 8192, C 192 103 / 67; P 120000, C 200 1375 / 869 (head_dim 64 1167 / 693); 16/2 heads, P 23838, C 599 240 / 165; 8/1 heads,
//     P 24084, C 1839 260 / 188.  When it is taken: plan_classes (host_plan.cpp).
//   * What bounds it at head_dim 128: the board's power limit.  7.0 % less time on all-zero operands,
//     which run at the full clock (128k-context shape, 2.58 -> 2.40 ms; 6.1 % fewer cycles by the
//     counters), came out as 1.3 % less on random ones (3.20 -> 3.16 ms): the clock falls as the stream
//     gets denser.  On one board: 1.36-1.37 PFLOP/s, where a large bf16 matrix product of the vendor
//     library reaches 1.37-1.40; on zeros both reach 1.78-1.80.
//   * At head_dim 64: the same vector work per block against half the MFMAs, 2.7 vector instructions
//     per MFMA where two are hidden; the matrix pipe is busy 50.5 % of the cycles (1.02 PFLOP/s).
#include <type_traits>

#include "attn_device.h"
#include "mc_internal.h"

namespace mc {
namespace {

typedef bf16x8 frag;
typedef f32x4 acc4;

// The reference of a row's probabilities is kept kRefLift (log2 units) ABOVE the largest score it was last set
// from, so probabilities are at most 2^-7 then and stay below 2 while later scores outgrow that maximum by less
// than 8: "some probability reached 2" is bit 14 of a bf16 pattern, which an OR over the block's packed
// probabilities finds (bit 14 is also set in inf and NaN).  The reference is raised when a score comes within
// kRaiseAbove of making its probability 2, which is before the guard can fire.
constexpr float kRefLift = 7.0f;
constexpr float kRaiseAbove = 0.5f;
constexpr uint32_t kGuardBits = 0x40004000u;

__device__ __forceinline__ acc4 mma(frag a, frag b, acc4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// Tile geometry for head_dim D (128: 256-byte rows, 64: 128-byte rows).
template <int D>
struct Geo {
  static_assert(D == 128 || D == 64, "head_dim");
  static constexpr int kRowB = D * 2;                    // bytes of a Q, K, V or O row
  static constexpr int kGran = kRowB / 16;               // 16-byte granules of a row
  static constexpr int kLineShift = D == 128 ? 0 : 1;    // log2 of the rows that share a 256-byte line of LDS banks
  static constexpr int kSteps = D / 32;                  // contraction steps of the scores over head_dim
  static constexpr int kDTiles = D / 16;                 // 16-column tiles of the output
  static constexpr int kRing = kDTiles;                  // K fragments of a block = V fragments of a block
  static_assert(kRing == 2 * kSteps, "both phases walk the ring once");
  static constexpr int kPageHeadB = kPageTokens * kRowB; // one (page, KV head), contiguous in the pool
  static constexpr int kKTileB = kTileKeys * kRowB;      // a K (or V) tile in LDS; rows dense, granules swizzled
  static constexpr int kChunkRows = 1024 / kRowB;        // rows one wave copy instruction (1 KiB) covers
  static constexpr int kPageChunks = kPageTokens / kChunkRows;

  // Order of a group of the pipeline (see weave): M = MFMA, L = ring refill, F = fma of a pair of scores, E = exp2 of
  // one, C = rounding of a pair.  At head_dim 128 a group has one pair of scores for four MFMAs, which hide about two
  // vector instructions each: the order below leaves the MFMAs of a step apart by the pair's fmas.  At head_dim 64 it
  // has two pairs for four MFMAs, more than they hide, and keeping the two MFMAs that share a fragment together wins.
  // Same box, all-zero operands (fixed clock: a cycle count) / random ones (power limit), 128k-context shape:
  //   head_dim 128   all vector work in the score phase, before its MFMAs (the form before)  2.58 / 3.20 ms
  //                  this order 2.40 / 3.16; eight other orders 2.48-2.62 / 3.20-3.26
  //   head_dim 64    the form before 1.89 ms / 0.714 ms (P 8189, C 4099); this order 1.76 / 0.691; eight others 1.80-1.86 / 0.697-0.706
  static constexpr char kOrder[] = "MFMLMEEMLC";
  static constexpr char kOrder64[] = "FEEMMLCFEEMMLC";

  // LDS swizzles: 16-byte granule g of tile row r is stored at granule g ^ swz(r).  The banks repeat every
  // 256 bytes, i.e. every row (D 128) or every second row (D 64).
  // K: a fragment read has 16 lanes on 16 consecutive rows at the same logical granule -> spread them over
  //    all 16 granule positions of a 256-byte line (D 64: two rows per line, 8 positions each).
  // V: a transpose read has 32 lanes on 8 consecutive rows x 32 bytes -> the 32-byte piece of a row moves
  //    with the line number, so the 8 rows cover all banks.
  static __device__ __forceinline__ int k_swz(int row) { return (row >> kLineShift) & (kGran - 1); }
  static __device__ __forceinline__ int v_swz(int row) { return ((row >> kLineShift) & (kGran / 2 - 1)) << 1; }

  // K fragment (key tile kt, head_dim step c) of a block: lane (j = l % 16, g = l / 16) reads
  // K[16 kt + j][32 c + 8 g .. + 7], i.e. granule 4 c + g of row 16 kt + j, stored at (4 c) ^ g ^ swz(j)
  // (the swizzle of row 16 kt + j is that of row j):  address = k_lane_off ^ (c << 6)  (+ row offset)
  static __device__ __forceinline__ int k_lane_off(int lane) {
    const int j = lane & 15, g = lane >> 4;
    return j * kRowB + ((g ^ k_swz(j)) << 4);
  }
  // ring slot i of a block's scores = (step i / 2, key tile i % 2)
  static __device__ __forceinline__ frag load_k(const uint32_t (&kx)[kSteps], int off, int i) {
    return *reinterpret_cast<MC_LDS const frag*>(kx[i >> 1] + off + (i & 1) * 16 * kRowB);
  }
  // V^T fragment (head_dim tile dt) of a block: lane (j, g) needs V[key][16 dt + j] for the keys 4 g + {0..3}
  // and 16 + 4 g + {0..3}.  The transpose read returns, to lane i of a 16-lane group, element i % 4 of
  // lanes i / 4, 4 + i / 4, 8 + i / 4, 12 + i / 4: source lane s addresses key 4 g + s / 4, columns
  // 16 dt + 4 (s % 4) .. + 3.  That is 8 bytes at byte 32 dt + 8 (s % 4) of row rr = 4 g + s / 4: 32-byte piece
  // dt, stored at piece dt ^ (v_swz(rr) / 2) (rows rr and rr + 16 swizzle alike):  address = v_lane_off ^ (dt << 5)
  static __device__ __forceinline__ int v_lane_off(int lane) {
    const int s = lane & 15, g = lane >> 4;
    const int rr = 4 * g + (s >> 2);
    return rr * kRowB + (v_swz(rr) << 4) + (((s & 3) >> 1) << 4) + ((s & 1) << 3);
  }
  static __device__ __forceinline__ frag load_v(const uint32_t (&vx)[kDTiles], int off, int dt) {
    const uint32_t p = vx[dt] + off;
    bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((MC_LDS bf16x4*)(uintptr_t)(p));
    bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((MC_LDS bf16x4*)(uintptr_t)(p + 16 * kRowB));
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  }
};

// largest of a value over the 4 lane groups that share a query row (lanes l, l ^ 16, l ^ 32, l ^ 48)
__device__ __forceinline__ float max_over_groups(float x) {
  x = fmaxf(x, __shfl_xor(x, 16, 64));
  return max_with_other_half(x);
}

// The scores of one 32-key block as a lane holds them: s[rt][kt] is the accumulator of score tile
// (key tile kt, row tile rt); its register r is key 16 kt + 4 g + r of the block, row 16 rt + j.
struct Scores {
  acc4 t[2][2];
  // e = 8 rt + 4 kt + r
  __device__ __forceinline__ float get(int e) const { return t[e >> 3][(e >> 2) & 1][e & 3]; }
  __device__ __forceinline__ void set(int e, float v) { t[e >> 3][(e >> 2) & 1][e & 3] = v; }
  __device__ __forceinline__ void zero() {
#pragma unroll
    for (int rt = 0; rt < 2; ++rt)
#pragma unroll
      for (int kt = 0; kt < 2; ++kt) t[rt][kt] = acc4{0.f, 0.f, 0.f, 0.f};
  }
};
// a block's probabilities as P V multiplies them: per row tile, the B operand of the 32-key step, kept as four
// words of two bf16 each (word k = keys 2 k, 2 k + 1 of the lane's eight)
struct PBlock {
  u32x4 w[2];
  __device__ __forceinline__ frag f(int rt) const { return __builtin_bit_cast(frag, w[rt]); }
};
typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;

// round probabilities e, e + 1 (same row tile) into their fragment
typedef float f32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t round_pair(const Scores& p, int e) {
  const f32x2 pp = {p.get(e), p.get(e + 1)};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(pp, bf16x2));      // one v_cvt_pk_bf16_f32 (round to nearest even)
}
template <int D, Rows ROWS, Form FORM>
__device__ __forceinline__ void attn_bf16_body(const AttnArgs& a, const Work& work) {
  constexpr bool SPLIT = FORM != kWhole;       // the result may be partial
  constexpr bool kByPairs = ROWS == kPairRows;   // every wave sees 32 of the 64 keys of a tile
  typedef Geo<D> X;
  // (these names hide the 256-byte-row constants of attn_device.h inside this kernel)
  constexpr int kD = D, kSteps = X::kSteps, kDTiles = X::kDTiles, kRing = X::kRing, kRowBytes = X::kRowB,
                kPageHeadBytes = X::kPageHeadB, kKTileBytes = X::kKTileB, kVTileBytes = X::kKTileB;
  // Tiles in LDS.  Two computing waves per SIMD keep the matrix pipe busy for longer than a copy takes: three buffers, a
  // tile's copy has one tile's time to land.  One is done with a tile sooner than its copy (launches of few rows stream K
  // and V at the memory's rate): four, two to three tiles in flight (16 tokens at 128k, 64/8 heads: 103.5 us a call with
  // three buffers, 97 with four or five; a short call, 1000 + 16 tokens: 16.9, 17.0, 17.4).
  constexpr int kBufs = ROWS == kFullRows ? kBuffers : kDeepBuffers;
  constexpr int kAhead = kBufs - 1;
  // Pair rows: a wave goes through a tile in one step, its scores run a tile ahead and their fragments one more, so K needs three
  // tiles where V needs one; with three and two more on their way that is 144 KiB (four buffers of V, 160 KiB and a loop of twelve
  // tiles: 1 % sooner).
  constexpr int kKBufs = kByPairs ? 6 : kBufs, kVBufs = kByPairs ? 3 : kBufs;
  constexpr int kVBase = kKBufs * kKTileBytes;           // the K tiles of the buffers, then the V tiles
  // tile bases are multiples of 8 KiB from a 256-byte aligned start: the XOR constants of the swizzle (< 256)
  // never reach a tile base
  __shared__ __attribute__((aligned(256))) char smem[kKBufs * kKTileBytes + kVBufs * kVTileBytes];
  constexpr int kTileRows = kTileRowsOf<ROWS>;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int g = lane >> 4;        // lane group: which 4 + 4 keys of a block
  const int j = lane & 15;        // row inside a row tile

  const int G = a.G;
  const int P = work.prefix;
  const int L = work.prefix + work.chunk;
  const int n_rows = work.chunk * G;
  const int last_page = (L - 1) / kPageTokens;

  // a wave that copies no tiles and whose 32 rows all lie past the end of the chunk ends here
  const int wave_u = __builtin_amdgcn_readfirstlane(wave);
  const bool fetcher = wave_copies<ROWS>(wave_u);
  const int row_wave = kByPairs ? wave & 1 : wave, row_wave_u = kByPairs ? wave_u & 1 : wave_u;
  const int key_half = kByPairs ? wave_u >> 1 & 1 : 0;
  if (!fetcher && work.row0 + row_wave_u * 32 >= n_rows) return;

  // ---- this lane's two query rows: their Q fragments stay in registers for the whole KV loop
  frag qf[kSteps][2];
  bool live[2];
  int tok[2];
  int64_t orow_idx[2], prow[2];                   // rows of the output and of the partial results
#pragma unroll
  for (int rt = 0; rt < 2; ++rt) {
    int row = work.row0 + row_wave * 32 + rt * 16 + j;
    live[rt] = row < n_rows;
    row = live[rt] ? row : n_rows - 1;            // dead rows recompute the last row, never stored
    tok[rt] = row / G;
    const int qhead = work.kv_head * G + (row - tok[rt] * G);
    orow_idx[rt] = (int64_t)(work.q_off + tok[rt]) * a.Hq + qhead;
    prow[rt] = work.part_row + (FORM == kClasses ? (int64_t)row : orow_idx[rt]);
    const char* qrow = reinterpret_cast<const char*>(a.q) + orow_idx[rt] * kRowBytes;
#pragma unroll
    for (int c = 0; c < kSteps; ++c) qf[c][rt] = *reinterpret_cast<const frag*>(qrow + c * 64 + g * 16);
  }

  // ---- keys this workgroup needs, and how many leading tiles need no mask
  const int tok_first = work.row0 / G;
  int tok_last = (work.row0 + kTileRows - 1) / G;
  tok_last = tok_last < work.chunk - 1 ? tok_last : work.chunk - 1;
  const int kv_end = P + tok_last + 1;                       // <= L
  int n_tiles = (kv_end + kTileKeys - 1) / kTileKeys;        // tiles [t_lo, n_tiles) are this item's
  int t_lo = 0;
  if (FORM == kSlices) {
    const int per = ((L + kTileKeys - 1) / kTileKeys + a.kv_splits - 1) / a.kv_splits;
    t_lo = work.piece * per;
    n_tiles = n_tiles < t_lo + per ? n_tiles : t_lo + per;
  }
  if (FORM == kClasses) piece_tiles(n_tiles, work.piece, work.pieces, &t_lo, &n_tiles);
  int n_free = (P + tok_first + 1) / kTileKeys;              // every key of these tiles is visible to every row
  n_free = n_free < n_tiles ? n_free : n_tiles;
  if (SPLIT && t_lo >= n_tiles) {
    // no key of the slice is visible to any row of the tile
#pragma unroll
    for (int rt = 0; rt < 2; ++rt)
      if (live[rt] && wave_computes<ROWS>(wave_u)) {
        char* orow = reinterpret_cast<char*>(a.o_parts) + prow[rt] * (kD * 4);
#pragma unroll
        for (int dt = 0; dt < kDTiles; ++dt)
          *reinterpret_cast<f32x4*>(orow + (dt * 16 + g * 4) * 4) = f32x4{0.f, 0.f, 0.f, 0.f};
        if (g == 0) a.lse_parts[prow[rt]] = -INFINITY;
      }
    return;
  }

  // ---- global -> LDS, no registers in between (as in attn_prefill.hip): one wave instruction writes
  //      1 KiB of LDS, 4 (D 64: 8) tile rows of 16 (8) granules inside one page; lane i fetches, for granule
  //      position i % kGran of row i / kGran, the logical granule (i % kGran) ^ swz(row).  One wave of each
  //      SIMD copies (which: see Rows), each one page of the tile: one page id, one page address and two LDS bases per tile,
  //      the chunks of the page are immediate offsets (they advance the global and the LDS address alike).
  static_assert(kFetchWaves == kTileKeys / kPageTokens, "one page of the tile per copying wave");
  const char* kbase = reinterpret_cast<const char*>(a.k_pool) + (int64_t)work.kv_head * kPageHeadBytes;
  const char* vbase = reinterpret_cast<const char*>(a.v_pool) + (int64_t)work.kv_head * kPageHeadBytes;
  const int64_t page_stride = (int64_t)a.Hkv * kPageHeadBytes;
  const int fetch_wave = wave_u & (kFetchWaves - 1);
  const uint32_t smem_base = (uint32_t)(uintptr_t)(MC_LDS char*)smem;
  typedef const __attribute__((address_space(4))) int32_t* const_i32_ptr;
  const_i32_ptr btc = (const_i32_ptr)(a.block_tables + (int64_t)work.req * a.max_pages);
  const int64_t first_page_off = (int64_t)btc[0] * page_stride;   // page of key 0: always valid
  int pid = 0, pid_next = 0;
  auto load_ids = [&](int tile) __attribute__((always_inline)) {
    if (!fetcher) return;
    const int lp = tile * (kTileKeys / kPageTokens) + fetch_wave;
    pid_next = btc[lp < last_page ? lp : last_page];         // never index the table past the request's pages
  };
  auto take_ids = [&]() __attribute__((always_inline)) { pid = pid_next; };
  uint32_t k_src[X::kPageChunks], v_src[X::kPageChunks];     // within a chunk
#pragma unroll
  for (int i = 0; i < X::kPageChunks; ++i) {
    const int row = i * X::kChunkRows + lane / X::kGran;
    k_src[i] = (uint32_t)(lane / X::kGran * kRowBytes + (((lane % X::kGran) ^ X::k_swz(row)) << 4));
    v_src[i] = (uint32_t)(lane / X::kGran * kRowBytes + (((lane % X::kGran) ^ X::v_swz(row)) << 4));
  }
  auto fetch = [&](int tile, int buf) __attribute__((always_inline)) {
    if (!fetcher) return;
    const uint32_t dst = smem_base + buf * kKTileBytes + fetch_wave * kPageHeadBytes;
    const int64_t page_off = (int64_t)pid * page_stride;
    if ((tile + 1) * kTileKeys <= L) {
      if (ROWS == kFewRows && work.once) {
        dma16_page<true>(kbase + page_off, k_src, dst);
        dma16_page<true>(vbase + page_off, v_src, dst + kVBase);
      } else {
        dma16_page<false>(kbase + page_off, k_src, dst);
        dma16_page<false>(vbase + page_off, v_src, dst + kVBase);
      }
    } else {
      // slots at or past the request's length may hold anything: those lanes copy row 0 of the request's
      // first page instead; the causal mask hides the key
#pragma unroll
      for (int i = 0; i < X::kPageChunks; ++i) {
        const int row = fetch_wave * kPageTokens + i * X::kChunkRows + lane / X::kGran;
        const bool in_seq = tile * kTileKeys + row < L;
        const char* ks = kbase + (in_seq ? page_off + i * 1024 + k_src[i] : first_page_off + (k_src[i] & (kRowBytes - 1)));
        const char* vs = vbase + (in_seq ? page_off + i * 1024 + v_src[i] : first_page_off + (v_src[i] & (kRowBytes - 1)));
        dma16(ks, dst + i * 1024);
        dma16(vs, dst + i * 1024 + kVBase);
      }
    }
  };
  // wait until all but the last `tiles` tiles this wave has enqueued have landed (vmcnt only)
  auto copies_landed = [&](auto tiles) __attribute__((always_inline)) {
    constexpr int n = decltype(tiles)::value * 2 * X::kPageChunks;
    static_assert(n < 64, "vmcnt");
    __builtin_amdgcn_s_waitcnt(0x0F70 | (n & 15) | (n >> 4 << 14));
  };

  // ---- running softmax state and output accumulators: o[dt][rt] register r = column 16 dt + 4 g + r of row 16 rt + j
  acc4 o[kDTiles][2];
  float m_run[2] = {-INFINITY, -INFINITY};   // reference of the probabilities accumulated so far (log2 units)
  float m_ref[2] = {kNoKeyYet, kNoKeyYet};   // the same as probabilities are formed with: finite
  // Row sums come from the matrix cores: l_acc[rt] += ones (16 x 32) . P^T (32 keys x 16 rows) leaves, in all four
  // registers of lane (j, g), the sum of row j's rounded probabilities over the whole block, lane groups included
  // (2 MFMAs per block instead of 8 dot-product instructions, which cost a matrix-pipe slot each).
  acc4 l_acc[2] = {acc4{0.f, 0.f, 0.f, 0.f}, acc4{0.f, 0.f, 0.f, 0.f}};
  frag ones;
#pragma unroll
  for (int e = 0; e < 8; ++e) ones[e] = (__bf16)1.0f;
  asm volatile("" : "+v"(ones));             // kept in registers, not rebuilt at every use
#pragma unroll
  for (int dt = 0; dt < kDTiles; ++dt)
#pragma unroll
    for (int rt = 0; rt < 2; ++rt) o[dt][rt] = acc4{0.f, 0.f, 0.f, 0.f};
  const float c = a.scale_log2e;
  const uint32_t k_lane = smem_base + key_half * 32 * kRowBytes + X::k_lane_off(lane);
  const uint32_t v_lane = smem_base + kVBase + key_half * 32 * kRowBytes + X::v_lane_off(lane);
  uint32_t kx[kSteps], vx[kDTiles];
#pragma unroll
  for (int i = 0; i < kSteps; ++i) kx[i] = k_lane ^ (uint32_t)(i << 6);
#pragma unroll
  for (int i = 0; i < kDTiles; ++i) vx[i] = v_lane ^ (uint32_t)(i << 5);

  // ---- building blocks that are NOT on the steady-state path (last blocks, rare recompute)
  auto qk_block = [&](int buf, int kb, Scores& s) __attribute__((always_inline)) {
    const int off = buf * kKTileBytes + kb * 32 * kRowBytes;
    s.zero();
#pragma unroll
    for (int i = 0; i < kRing; ++i) {
      const frag kf = X::load_k(kx, off, i);
      s.t[0][i & 1] = mma(kf, qf[i >> 1][0], s.t[0][i & 1]);
      s.t[1][i & 1] = mma(kf, qf[i >> 1][1], s.t[1][i & 1]);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // Mask a block if it reaches the diagonal, take the TRUE row maxima and raise the references if some row
  // outgrew its own by more than the slack (rare, wave-uniform branch; always taken for the first block).
  auto settle_reference = [&](Scores& s, int key0, auto masked_tag) __attribute__((always_inline)) {
    constexpr bool kMasked = decltype(masked_tag)::value;
    float mx[2];
#pragma unroll
    for (int rt = 0; rt < 2; ++rt) {
      if (kMasked) {
        // key of (kt, r): key0 + 16 kt + 4 g + r; visible iff <= P + tok
        const int lim = P + tok[rt] - key0 - 4 * g;
#pragma unroll
        for (int kt = 0; kt < 2; ++kt)
#pragma unroll
          for (int r = 0; r < 4; ++r) s.t[rt][kt][r] = (16 * kt + r <= lim) ? s.t[rt][kt][r] : -INFINITY;
      }
      float m = s.t[rt][0][0];
#pragma unroll
      for (int e = 1; e < 8; ++e) m = fmaxf(m, s.t[rt][e >> 2][e & 3]);
      mx[rt] = max_over_groups(m) * c;
    }
    if (__builtin_amdgcn_ballot_w64(mx[0] > m_run[0] + kRaiseAbove || mx[1] > m_run[1] + kRaiseAbove) != 0) {
#pragma unroll
      for (int rt = 0; rt < 2; ++rt) {
        const float m_new = fmaxf(m_run[rt], mx[rt] + kRefLift);
        // a row that has seen no key yet keeps -inf (only in a slice that starts beyond the row's diagonal, or in the later keys
        // of a tile)
        const float alpha = ((SPLIT || kByPairs) && m_new == -INFINITY) ? 1.f : __builtin_amdgcn_exp2f(m_run[rt] - m_new);
        l_acc[rt] *= alpha;
        m_run[rt] = m_new;
        m_ref[rt] = SPLIT || kByPairs ? fmaxf(m_new, kNoKeyYet) : m_new;
#pragma unroll
        for (int dt = 0; dt < kDTiles; ++dt) o[dt][rt] *= alpha;
      }
    }
  };
  // scores -> probabilities against the references as they stand, rounded the way P V multiplies them
  auto probabilities = [&](Scores& s, PBlock& pb) __attribute__((always_inline)) {
#pragma unroll
    for (int rt = 0; rt < 2; ++rt) {
#pragma unroll
      for (int e = 8 * rt; e < 8 * rt + 8; ++e) s.set(e, __builtin_amdgcn_exp2f(__builtin_fmaf(s.get(e), c, -m_ref[rt])));
#pragma unroll
      for (int k = 0; k < 4; ++k) pb.w[rt][k] = round_pair(s, 8 * rt + 2 * k);
    }
  };
  auto add_row_sums = [&](const PBlock& pb) __attribute__((always_inline)) {
    l_acc[0] = mma(ones, pb.f(0), l_acc[0]);
    l_acc[1] = mma(ones, pb.f(1), l_acc[1]);
  };

  // ---- KV loop.  Software pipeline over 32-key blocks, scheduled by hand (the order written is the order
  //      issued), around one ring of 8 fragment registers:
  //        phase A  scores of block j+1: step i multiplies ring[i] (K fragment i, read during the previous
  //                 phase B) into both row tiles and frees it; the V fragment that P V step i of block j
  //                 needs is read into the freed slot; under these MFMAs the vector ALU turns the scores of
  //                 block j, row tile 1, into probabilities.
  //        phase B  P V of block j: step i multiplies ring[i] (the V fragment) into both row tiles and frees
  //                 it; K fragment i of block j+2 is read into the freed slot; under these MFMAs the scores of
  //                 block j+1, row tile 0, become probabilities.  (The last block the pipeline leaves scores of
  //                 is one of those that may reach the diagonal: its scores are computed again, row tile 0 of
  //                 them is overwritten by then.)
  frag ring[kRing];
  Scores s_cur, s_next;
  auto load_k_ring = [&](int buf, int kb) __attribute__((always_inline)) {
    const int off = buf * kKTileBytes + kb * 32 * kRowBytes;
#pragma unroll
    for (int i = 0; i < kRing; ++i) ring[i] = X::load_k(kx, off, i);
  };
  // a probability of 2 or more (or not finite) means its score outgrew the reference: the block is then
  // recomputed against its true maxima (nothing was accumulated yet)
  PBlock pb;
  u32x4 pb_ahead;                        // rounded probabilities of row tile 0 of the block whose scores are in s_next
  // One group of a phase in the order Geo prescribes: four MFMAs (two steps of the ring, consecutive ones sharing an
  // operand register), the refill of their two ring slots and the vector work that turns kPairs pairs of scores of row
  // tile rt into rounded probabilities.
  constexpr int kPairs = 8 / kRing;
  constexpr int kOps = (D == 128 ? sizeof(X::kOrder) : sizeof(X::kOrder64)) - 1;
  auto weave = [&](auto&& mfma, auto&& refill, Scores& s, u32x4& w, int rt, int grp) __attribute__((always_inline)) {
    const int e0 = 8 * rt + 2 * kPairs * grp;
    int m = 0, l = 0, f = 0, x = 0, k = 0;
#pragma unroll
    for (int t = 0; t < kOps; ++t) {
      const char op = D == 128 ? X::kOrder[t] : X::kOrder64[t];
      if (op == 'M') {
        mfma(2 * grp + (m >> 1), (m == 1 || m == 2) ? 1 : 0);
        ++m;
      } else if (op == 'L') {
        refill(2 * grp + l);
        ++l;
      } else if (op == 'F') {
        s.set(e0 + 2 * f, __builtin_fmaf(s.get(e0 + 2 * f), c, -m_ref[rt]));
        s.set(e0 + 2 * f + 1, __builtin_fmaf(s.get(e0 + 2 * f + 1), c, -m_ref[rt]));
        ++f;
      } else if (op == 'E') {
        s.set(e0 + x, __builtin_amdgcn_exp2f(s.get(e0 + x)));
        ++x;
      } else {
        w[kPairs * grp + k] = round_pair(s, e0 + 2 * k);
        ++k;
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  auto phase_a = [&](int buf_cur, int kb_cur) __attribute__((always_inline)) {
    const int off_v = buf_cur % kVBufs * kVTileBytes + kb_cur * 32 * kRowBytes;
    s_cur = s_next;
    s_next.zero();
    pb.w[0] = pb_ahead;
    auto score = [&](int i, int rt) __attribute__((always_inline)) {
      s_next.t[rt][i & 1] = mma(ring[i], qf[i >> 1][rt], s_next.t[rt][i & 1]);
      __builtin_amdgcn_sched_barrier(0);
    };
    auto refill = [&](int i) __attribute__((always_inline)) {
      ring[i] = X::load_v(vx, off_v, i);
      __builtin_amdgcn_sched_barrier(0);
    };
#pragma unroll
    for (int grp = 0; grp < kRing / 2; ++grp) {
      weave(score, refill, s_cur, pb.w[1], 1, grp);
    }
    // OR of the block's packed probabilities
    const uint32_t seen = pb.w[0][0] | pb.w[0][1] | pb.w[0][2] | pb.w[0][3] | pb.w[1][0] | pb.w[1][1] | pb.w[1][2] | pb.w[1][3];
    if (__builtin_expect(__builtin_amdgcn_ballot_w64((seen & kGuardBits) != 0) != 0, 0)) {   // (laid out behind the loop)
      qk_block(buf_cur, kb_cur, s_cur);
      settle_reference(s_cur, 0, std::false_type{});
      probabilities(s_cur, pb);
    }
  };
  auto phase_b = [&](int buf_pre, int kb_pre) __attribute__((always_inline)) {
    const int off_k = buf_pre * kKTileBytes + kb_pre * 32 * kRowBytes;
    auto accumulate = [&](int i, int rt) __attribute__((always_inline)) {
      o[i][rt] = mma(ring[i], pb.f(rt), o[i][rt]);
      __builtin_amdgcn_sched_barrier(0);
      if (i < 2 && rt == (i & 1)) {        // the row sums of the tile just used: the P operand stays where it is
        l_acc[rt] = mma(ones, pb.f(rt), l_acc[rt]);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    auto refill = [&](int i) __attribute__((always_inline)) {
      ring[i] = X::load_k(kx, off_k, i);
      __builtin_amdgcn_sched_barrier(0);
    };
#pragma unroll
    for (int grp = 0; grp < kRing / 2; ++grp) {
      weave(accumulate, refill, s_next, pb_ahead, 0, grp);
    }
  };
  // One block start to finish, for the few blocks that may reach the diagonal: the ring is free there, so the block's K
  // fragments are read together, and its V fragments under the softmax.  (A fragment read just before its MFMAs cost its
  // whole latency: one call, P 256, C 128, 64/8 heads 13.4 us, now 12.8; P 1000, C 16 17.0, 16.2.)
  auto scores_of = [&](int buf, int kb, Scores& s) __attribute__((always_inline)) {
    load_k_ring(buf, kb);
    s.zero();
#pragma unroll
    for (int i = 0; i < kRing; ++i) {
      s.t[0][i & 1] = mma(ring[i], qf[i >> 1][0], s.t[0][i & 1]);
      s.t[1][i & 1] = mma(ring[i], qf[i >> 1][1], s.t[1][i & 1]);
    }
  };
  auto plain_block = [&](int buf, int kb, int key0, Scores& s, bool have_scores) __attribute__((always_inline)) {
    if (!have_scores) scores_of(buf, kb, s);
    const int off = (kByPairs ? buf % kVBufs : buf) * kVTileBytes + kb * 32 * kRowBytes;
#pragma unroll
    for (int dt = 0; dt < kDTiles; ++dt) ring[dt] = X::load_v(vx, off, dt);
    settle_reference(s, key0, std::true_type{});
    PBlock pbl;
    probabilities(s, pbl);
    add_row_sums(pbl);
#pragma unroll
    for (int dt = 0; dt < kDTiles; ++dt) {
      o[dt][0] = mma(ring[dt], pbl.f(0), o[dt][0]);
      o[dt][1] = mma(ring[dt], pbl.f(1), o[dt][1]);
    }
  };

  // The copies of the first tiles; everything enqueued so far (also the Q fragments) has landed, those of the rest of the
  // buffers are on their way.
  auto first_copies = [&]() __attribute__((always_inline)) {
    load_ids(t_lo);
    take_ids();
    fetch(t_lo, 0);
    load_ids(t_lo + 1);
    take_ids();
    if (n_tiles > t_lo + 1) {
      fetch(t_lo + 1, 1);
      load_ids(t_lo + 2);
      take_ids();
    }
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
#pragma unroll
    for (int i = 2; i < kAhead; ++i)
      if (n_tiles > t_lo + i) {
        fetch(t_lo + i, i);
        load_ids(t_lo + i + 1);
        take_ids();
      }
  };
  // Tile `tile` begins: the copy of the next one has landed everywhere (the scores run a block ahead), the buffer of the
  // one before is free and takes tile + kAhead, whose ids were loaded a tile ago.
  int buf = 0;
  // Pair rows: what the waves that copy do.  When tile t begins, K of tile t + 2 and V of tile t have landed everywhere, and the
  // buffers of tile t - 1 are free: they take K of tile t + 5 and V of tile t + 2.
  auto copy_pair_tiles = [&]() __attribute__((always_inline)) {
    auto ids_of = [&](int tile) __attribute__((always_inline)) {
      const int lp = tile * (kTileKeys / kPageTokens) + fetch_wave;
      return (int)btc[lp < last_page ? lp : last_page];
    };
    // one half of a tile's copies: K or V
    auto fetch_half = [&](const char* base, const uint32_t (&src)[X::kPageChunks], uint32_t tiles_at, int tile, int id) __attribute__((always_inline)) {
      const uint32_t dst = smem_base + tiles_at + fetch_wave * kPageHeadBytes;
      const int64_t page_off = (int64_t)id * page_stride;
      if ((tile + 1) * kTileKeys <= L) {
        dma16_page<false>(base + page_off, src, dst);
      } else {
#pragma unroll
        for (int i = 0; i < X::kPageChunks; ++i) {           // (see fetch)
          const int row = fetch_wave * kPageTokens + i * X::kChunkRows + lane / X::kGran;
          const bool in_seq = tile * kTileKeys + row < L;
          dma16(base + (in_seq ? page_off + i * 1024 + src[i] : first_page_off + (src[i] & (kRowBytes - 1))), dst + i * 1024);
        }
      }
    };
    auto fetch_k = [&](int tile, int b, int id) __attribute__((always_inline)) {
      if (tile < n_tiles) fetch_half(kbase, k_src, b * kKTileBytes, tile, id);
    };
    auto fetch_v = [&](int tile, int b, int id) __attribute__((always_inline)) {
      if (tile < n_tiles) fetch_half(vbase, v_src, kVBase + b * kVTileBytes, tile, id);
    };
    int id[6];
#pragma unroll
    for (int i = 0; i < 6; ++i) id[i] = ids_of(t_lo + i);
    fetch_k(t_lo, 0, id[0]);
    fetch_v(t_lo, 0, id[0]);
    fetch_k(t_lo + 1, 1, id[1]);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    fetch_k(t_lo + 2, 2, id[2]);
    fetch_v(t_lo + 1, 1, id[1]);
    fetch_k(t_lo + 3, 3, id[3]);
    fetch_k(t_lo + 4, 4, id[4]);
    int v_id = id[2], id_3 = id[3], id_4 = id[4], k_id = id[5], k_buf = 5, v_buf = 2;
    for (int tile = t_lo; tile < n_tiles; ++tile) {
      const int next_id = ids_of(tile + 6);
      // enqueued last: K of tile + 4 and V of tile + 1, as far as there are such tiles (at the start K of the tiles before, too)
      constexpr int kHalf = X::kPageChunks;
      if (tile + 4 < n_tiles) __builtin_amdgcn_s_waitcnt(0x0F70 | 2 * kHalf);
      else if (tile + 1 < n_tiles) __builtin_amdgcn_s_waitcnt(0x0F70 | kHalf);
      else __builtin_amdgcn_s_waitcnt(0x0F70);
      __syncthreads();
      fetch_k(tile + 5, k_buf, k_id);
      fetch_v(tile + 2, v_buf, v_id);
      v_id = id_3;
      id_3 = id_4;
      id_4 = k_id;
      k_id = next_id;
      k_buf = k_buf == kKBufs - 1 ? 0 : k_buf + 1;
      v_buf = v_buf == kVBufs - 1 ? 0 : v_buf + 1;
    }
  };
  auto copy_sync = [&](int tile) __attribute__((always_inline)) {
    const bool ahead = tile + kAhead < n_tiles;
    if (ahead) load_ids(tile + kAhead + 1);
    // enqueued so far: tiles up to tile + kAhead - 1, as far as there are any
    if (kAhead > 2 && tile + kAhead - 1 < n_tiles) copies_landed(std::integral_constant<int, kAhead - 2>{});
    else copies_landed(std::integral_constant<int, 0>{});
    __syncthreads();
    if (ahead) {
      fetch(tile + kAhead, buf == 0 ? kBufs - 1 : buf - 1);
      take_ids();
    }
  };
  auto tile_sync = [&](int tile) __attribute__((always_inline)) {
    if constexpr (ROWS == kFullRows) copy_sync(tile);
    else __syncthreads();
  };
  if constexpr (kByPairs) {
    if (fetcher) {
      copy_pair_tiles();
      return;
    }
    __syncthreads();
  } else if constexpr (ROWS == kFewRows) {
    if (fetcher) {
      first_copies();
      for (int tile = t_lo; tile < n_tiles; ++tile) {
        copy_sync(tile);
        buf = buf == kBufs - 1 ? 0 : buf + 1;
      }
      return;
    }
    __syncthreads();
  } else {
    first_copies();
  }
  int tile = t_lo;
  const int n_plain = n_free < n_tiles - 1 ? n_free : n_tiles - 1;
  scores_of(0, 0, s_next);
  if (tile < n_plain) {
    settle_reference(s_next, 0, std::false_type{});
    if constexpr (kByPairs) load_k_ring(1, 0);
    else load_k_ring(0, 1);
#pragma unroll
    for (int e = 0; e < 8; ++e) s_next.set(e, __builtin_amdgcn_exp2f(__builtin_fmaf(s_next.get(e), c, -m_ref[0])));
#pragma unroll
    for (int k = 0; k < 4; ++k) pb_ahead[k] = round_pair(s_next, 2 * k);
    // the two waves of a SIMD run half a step apart (see attn_prefill.hip)
    // (few rows: the waves that would be late only copy.  The compiler is not told: with the barrier unconditional the
    // phases become one basic block, in which it keeps 28 registers too many alive and spills 52.)
    int w = wave_u;
    if constexpr (ROWS != kFullRows) asm volatile("" : "+s"(w));
    const bool late_barrier = w >= kFetchWaves;
    auto pipelined_tile = [&](auto buf_tag) __attribute__((always_inline)) {
      constexpr int b = decltype(buf_tag)::value, bn = (b + 1) % kBufs;
      if constexpr (kByPairs) {
        buf = b;
        if (!late_barrier) tile_sync(tile);
        phase_a(b, 0);
        if (late_barrier) tile_sync(tile);
        phase_b((b + 2) % kKBufs, 0);
        buf = (b + 1) % kKBufs;
        ++tile;
        return;
      }
      buf = b;
      if (!late_barrier) tile_sync(tile);
      phase_a(b, 0);
      if (late_barrier) tile_sync(tile);
      phase_b(bn, 0);
      phase_a(b, 1);
      phase_b(bn, 1);
      buf = bn;
      ++tile;
    };
    for (;;) {
      if (tile >= n_plain) break;
      // Where the loop body sits relative to the 64-byte instruction fetch lines changes its speed by up to
      // 3.5 % (all 16 offsets measured on the 128k-context workload, with the rare recompute path laid out
      // behind the loop); pin the best one, so that edits elsewhere in the kernel cannot move it.
      asm volatile(".p2align 6");
      pipelined_tile(std::integral_constant<int, 0>{});
      if (tile >= n_plain) break;
      pipelined_tile(std::integral_constant<int, 1>{});
      if (tile >= n_plain) break;
      pipelined_tile(std::integral_constant<int, 2>{});
      if constexpr (kKBufs >= 4) {
        if (tile >= n_plain) break;
        pipelined_tile(std::integral_constant<int, 3>{});
      }
      if constexpr (kKBufs == 6) {
        if (tile >= n_plain) break;
        pipelined_tile(std::integral_constant<int, 4>{});
        if (tile >= n_plain) break;
        pipelined_tile(std::integral_constant<int, 5>{});
      }
    }
  }
  bool have_scores = n_plain <= t_lo;
  for (; tile < n_tiles; ++tile) {
    const int buf_next = buf == kKBufs - 1 ? 0 : buf + 1;
    tile_sync(tile);
    plain_block(buf, 0, tile * kTileKeys + key_half * 32, s_next, have_scores);
    have_scores = false;
    if constexpr (!kByPairs) plain_block(buf, 1, tile * kTileKeys + 32, s_next, false);
    buf = buf_next;
  }

  // ---- pair rows: the other pair's references, sums and outputs of the same rows, lane by lane through LDS
  if constexpr (kByPairs) {
    constexpr int kLaneB = (kDTiles * 2 + 1) * 16;           // bytes of a lane: its output, and (m, l) of both row tiles
    static_assert(2 * 64 * kLaneB <= sizeof(smem), "room for two waves");
    char* const mine = smem + row_wave_u * (64 * kLaneB) + lane * 16;
    __syncthreads();                                         // (the tiles are done with)
    if (key_half == 1) {
#pragma unroll
      for (int dt = 0; dt < kDTiles; ++dt)
#pragma unroll
        for (int rt = 0; rt < 2; ++rt) *reinterpret_cast<acc4*>(mine + (2 * dt + rt) * 1024) = o[dt][rt];
      *reinterpret_cast<acc4*>(mine + 2 * kDTiles * 1024) = acc4{m_run[0], l_acc[0][0], m_run[1], l_acc[1][0]};
    }
    __syncthreads();
    if (key_half == 1) return;
    const acc4 other = *reinterpret_cast<const acc4*>(mine + 2 * kDTiles * 1024);
#pragma unroll
    for (int rt = 0; rt < 2; ++rt) {
      const float top = fmaxf(m_run[rt], other[2 * rt]), ref = top == -INFINITY ? 0.f : top;
      const float here = __builtin_amdgcn_exp2f(m_run[rt] - ref), there = __builtin_amdgcn_exp2f(other[2 * rt] - ref);
      m_run[rt] = top;
      l_acc[rt][0] = l_acc[rt][0] * here + other[2 * rt + 1] * there;
#pragma unroll
      for (int dt = 0; dt < kDTiles; ++dt)
        o[dt][rt] = o[dt][rt] * here + *reinterpret_cast<const acc4*>(mine + (2 * dt + rt) * 1024) * there;
    }
  }

  // ---- epilogue: normalise, round, store; a lane holds 4 consecutive columns per (dt, rt)
#pragma unroll
  for (int rt = 0; rt < 2; ++rt) {
    const float l_run = l_acc[rt][0];
    if (!live[rt]) continue;
    if (FORM == kWhole || (FORM == kClasses && work.pieces == 1)) {
      const float inv = 1.0f / l_run;
      char* orow = reinterpret_cast<char*>(a.out) + orow_idx[rt] * kRowBytes;
#pragma unroll
      for (int dt = 0; dt < kDTiles; ++dt) {
        bf16x4 v;
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = (__bf16)(o[dt][rt][r] * inv);
        *reinterpret_cast<bf16x4*>(orow + (dt * 16 + g * 4) * 2) = v;
      }
      if (a.lse != nullptr && g == 0)
        a.lse[orow_idx[rt]] = (m_run[rt] + __builtin_amdgcn_logf(l_run)) * 0.6931471805599453f;
    } else {
      // partial result in fp32; a row that saw no key of the slice has l = 0: zeros and -inf (and nothing else has: a NaN
      // stays one)
      const bool no_key = l_run == 0.f;
      const float inv = no_key ? 0.f : 1.0f / l_run;
      char* orow = reinterpret_cast<char*>(a.o_parts) + prow[rt] * (kD * 4);
#pragma unroll
      for (int dt = 0; dt < kDTiles; ++dt)
        *reinterpret_cast<f32x4*>(orow + (dt * 16 + g * 4) * 4) =
            f32x4{o[dt][rt][0] * inv, o[dt][rt][1] * inv, o[dt][rt][2] * inv, o[dt][rt][3] * inv};
      if (g == 0)
        a.lse_parts[prow[rt]] =
            no_key ? -INFINITY : (m_run[rt] + __builtin_amdgcn_logf(l_run)) * 0.6931471805599453f;
    }
  }
}

template <int D, Rows ROWS, bool SPLIT>
__global__ __launch_bounds__(kWaves * 64) void attn_prefill_bf16_kernel(const AttnArgs a) {
  const Work work = work_of<ROWS>(a, blockIdx.x);
  if (ROWS != kFullRows && work.row0 >= work.chunk * a.G) return;     // a second half (later quarter) without rows
  attn_bf16_body<D, ROWS, SPLIT ? kSlices : kWhole>(a, work);
}

template <int D, Rows ROWS>
__global__ __launch_bounds__(kWaves * 64) void attn_prefill_bf16_classes_kernel(const AttnArgs a, const AttnClasses t) {
  attn_bf16_body<D, ROWS, kClasses>(a, work_of<kTileRowsOf<ROWS>>(t, blockIdx.x, a.Hkv, a.G));
}

}  // namespace

template <int D, Rows ROWS>
static void enqueue_list(const AttnArgs& args, hipStream_t stream) {
  const int wgs = ROWS == kPairRows ? args.n_items * (kAttnTileRows / kAttnPairRows) : args.n_items << args.halves;
  if constexpr (ROWS == kPairRows) attn_prefill_bf16_kernel<D, ROWS, false><<<wgs, kWaves * 64, 0, stream>>>(args);
  else if (args.kv_splits > 0) attn_prefill_bf16_kernel<D, ROWS, true><<<wgs, kWaves * 64, 0, stream>>>(args);
  else attn_prefill_bf16_kernel<D, ROWS, false><<<wgs, kWaves * 64, 0, stream>>>(args);
}
template <int D, Rows ROWS>
static void enqueue_classes(const AttnArgs& args, const AttnClasses& t, hipStream_t stream) {
  attn_prefill_bf16_classes_kernel<D, ROWS><<<args.n_items, kWaves * 64, 0, stream>>>(args, t);
}

hipError_t launch_attn_bf16_classes(const AttnArgs& args, const AttnClasses& t, hipStream_t stream) {
  (void)hipGetLastError();
  const bool few = t.rows == kAttnFewRows, pairs = t.rows == kAttnPairRows;
  if (pairs && args.head_dim == 128) enqueue_classes<128, kPairRows>(args, t, stream);
  else if (pairs && args.head_dim == 64) enqueue_classes<64, kPairRows>(args, t, stream);
  else if (args.head_dim == 128) few ? enqueue_classes<128, kFewRows>(args, t, stream) : enqueue_classes<128, kFullRows>(args, t, stream);
  else if (args.head_dim == 64) few ? enqueue_classes<64, kFewRows>(args, t, stream) : enqueue_classes<64, kFullRows>(args, t, stream);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_attn_bf16(const AttnArgs& args, hipStream_t stream) {
  (void)hipGetLastError();   // drop any stale error of earlier, unrelated runtime calls
  if (args.pair_rows && args.head_dim == 128) enqueue_list<128, kPairRows>(args, stream);
  else if (args.pair_rows && args.head_dim == 64) enqueue_list<64, kPairRows>(args, stream);
  else if (args.head_dim == 128) args.few_rows ? enqueue_list<128, kFewRows>(args, stream) : enqueue_list<128, kFullRows>(args, stream);
  else if (args.head_dim == 64) args.few_rows ? enqueue_list<64, kFewRows>(args, stream) : enqueue_list<64, kFullRows>(args, stream);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace mc
