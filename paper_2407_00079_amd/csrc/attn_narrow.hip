// Narrow form of the attention kernels: a workgroup owns 32 (fp32, or no more of them: 16) stacked query rows of one (request,
// KV head) and its eight waves share out the KEYS of those rows, each walking every eighth 32-key block by itself; their
// results meet in LDS once, at the end (paper Section 5.1: attention is associative over key slices).
//
// The other forms give each wave rows of its own, 128 or 256 a workgroup, and all of them every key: a launch of few rows
// leaves most of the chip idle and walks its keys at the pace of one workgroup.  Here a workgroup walks them at the rate one
// compute unit can load them.  No partial results in memory, so it is what callers without room for them run (prepared
// plans, calls without a workspace, calls with the minimal one), and no merge launch, which short calls gain from.  Where there
// is room its row tiles are cut into pieces as those of the other forms are, into fewer: a workgroup starts sooner (4.7 us with
// its launch, 7.6 the 128-row form) and a piece of four key tiles takes about as long as one of a single tile.
//
//   * A wave's block is its own: no barrier in the loop, and no tile that others wait for.  K and V go from the pool to
//     registers, the next block's K while this one's scores are formed, its V as soon as P V has let go of this one's; K is
//     turned into fragments in the wave's own corner of LDS.
//   * S^T = K Q^T and O^T += V^T P^T on the tiles of the other kernels (16x16x32; fp32 16x16x4).  V needs no turning: output
//     tile e holds the columns kVec i + e, so the kVec consecutive columns of a V row that a lane loads are one element of each
//     tile.  bf16: the eight keys of a contraction come from eight registers, two at a time by v_perm; fp32: a register is an
//     operand.
//   * Where the row tiles leave most of the chip idle, several workgroups take a row tile, each a share of the output's columns: all
//     of K, all scores and probabilities, its share of V and of P V.  Every column is summed as it is by one workgroup, so the
//     results are the same bits.  Which: narrow_shares (host_plan.cpp).
//   * True maxima per block, reference raised when a score outgrows it by 8 log2 units (see attn_prefill.hip).
//
// What bounds it: the loads of one compute unit (16 KiB in flight a wave).  One workgroup a compute unit, us a 64-key tile,
// against the 128-row form's: bf16 head_dim 128 0.30 (108 GB/s) / 0.67, head_dim 64 0.21 / 0.56, fp32 0.58 (of it 0.43 MFMA)
// / 3.8.  Lanes that load their K fragments themselves read 16 rows in a quarter wave: 0.545 us.  Loads behind a branch (no next
// block, the last block's slots past the end) make the compiler wait for all loads in flight before V is used: 0.33.  The nt
// hint: 0.53.  64 keys a block (head_dim 64): no change; two workgroups a compute unit (128 registers): 0.27 and fp32 0.73.
// Whole calls before / now, us: planned, 64/8 heads, P 30000, C 90 350 / 148; P 131056, C 16 1490 / 908; 16/16 heads, P 7206,
// C 200 93 / 41; head_dim 64, 64/8 heads, P 30000, C 90 301 / 104; fp32, 8/2 heads, P 2798, C 62 183 / 31; one call with room
// for pieces, fp32, 4/1 heads, P 256, C 128, append included, both calls through ctypes: 18.8 / 14.2.  450 random one-shot calls whose narrow row tiles may
// be cut, against only whole ones: geometric mean x1.05 (fp32 x1.25), the slowest x0.96.  When it is taken: plan_classes
// (host_plan.cpp).
#include "attn_device.h"
#include "mc_internal.h"

namespace mc {
namespace {

// What both dtypes share: a wave's corner of LDS and the meeting of the eight waves.
template <int ROWS, int D, int SPLIT, int BLOCK_KEYS, typename Out>
struct Narrow {
  static constexpr int kCols = D / SPLIT;                  // columns of the workgroup's share of the output
  static constexpr int kStride = kCols + 4;                // floats from row to row in LDS: 16 rows of a column spread over the banks
  // A wave's corner holds its block of keys in turn and, when it is done with them, its unnormalised output.
  static constexpr int kKeyBytes = BLOCK_KEYS * D * (int)sizeof(Out), kOutBytes = ROWS * kStride * 4;
  static constexpr int kCorner = ((kKeyBytes > kOutBytes ? kKeyBytes : kOutBytes) + 255) & ~255;
  struct Shared {
    char corner[kWaves][kCorner];
    float m[kWaves][ROWS], l[kWaves][ROWS];
    __device__ __forceinline__ const float* o(int wave, int row) const {
      return reinterpret_cast<const float*>(corner[wave]) + row * kStride;
    }
    __device__ __forceinline__ float* o(int wave, int row) { return reinterpret_cast<float*>(corner[wave]) + row * kStride; }
  };
  // Rows row0 .. of the chunk, columns share kCols .., over the waves' references, sums and unnormalised outputs in sh.
  static __device__ __forceinline__ void finish(const Shared& sh, const AttnArgs& a, const Work& work, int share, int n_rows) {
    constexpr int kShare = ROWS * kCols / (kWaves * 64), kPer = kShare > 0 ? kShare : 1;       // columns of a thread
    const int row = threadIdx.x / (kCols / kPer), col = threadIdx.x % (kCols / kPer) * kPer, out_col = share * kCols + col;
    if ((kShare == 0 && row >= ROWS) || work.row0 + row >= n_rows) return;
    float top = sh.m[0][row];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) top = fmaxf(top, sh.m[w][row]);
    // (no wave has a key for the row: in a piece of the keys, or where every score is -inf or NaN)
    const float ref = top == -INFINITY ? 0.f : top;
    float l = 0.f, acc[kPer];
#pragma unroll
    for (int e = 0; e < kPer; ++e) acc[e] = 0.f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      const float weight = __builtin_amdgcn_exp2f(sh.m[w][row] - ref);      // 0 for a wave without keys
      l += weight * sh.l[w][row];
#pragma unroll
      for (int e = 0; e < kPer; ++e) acc[e] += weight * sh.o(w, row)[col + e];
    }
    const int at = work.row0 + row, tok = at / a.G;
    const int64_t dst = (int64_t)(work.q_off + tok) * a.Hq + work.kv_head * a.G + (at - tok * a.G);
    if (work.pieces > 1) {
      // partial result in fp32; a row that saw no key of the piece has l = 0: zeros and -inf
      const float inv = l == 0.f ? 0.f : 1.0f / l;
      const int64_t part = work.part_row + at;
      float v __attribute__((ext_vector_type(kPer)));
#pragma unroll
      for (int e = 0; e < kPer; ++e) v[e] = acc[e] * inv;
      *reinterpret_cast<decltype(v)*>(a.o_parts + part * D + out_col) = v;
      if (out_col == 0) a.lse_parts[part] = l == 0.f ? -INFINITY : (top + __builtin_amdgcn_logf(l)) * 0.6931471805599453f;
      return;
    }
    const float inv = 1.0f / l;
    Out v __attribute__((ext_vector_type(kPer)));
#pragma unroll
    for (int e = 0; e < kPer; ++e) v[e] = (Out)(acc[e] * inv);
    *reinterpret_cast<decltype(v)*>(reinterpret_cast<Out*>(a.out) + dst * D + out_col) = v;
    if (a.lse != nullptr && out_col == 0) a.lse[dst] = (top + __builtin_amdgcn_logf(l)) * 0.6931471805599453f;
  }
};

__device__ __forceinline__ f32x4 mma(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x4 mma(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

// A NaN stays one (and raises no reference); fmaxf would cost a second instruction each to quieten what it then drops.
__device__ __forceinline__ float larger(float a, float b) { return __builtin_elementwise_maximum(a, b); }
// largest of a value over the 4 lane groups that share a query row: rows of 16 lanes exchanged in registers, as halves are
__device__ __forceinline__ float max_over_groups(float x) {
  float a = x, b = x;
  asm volatile("s_nop 1\n\tv_permlane16_swap_b32 %0, %1\n\ts_nop 1" : "+v"(a), "+v"(b));
  a = b = larger(a, b);
  swap_halves(a, b);
  return larger(a, b);
}
__device__ __forceinline__ float max8(f32x4 a, f32x4 b) {
  float m = a[0];
#pragma unroll
  for (int e = 1; e < 8; ++e) m = larger(m, e < 4 ? a[e] : b[e - 4]);
  return m;
}

// Between one lane's write of LDS and another lane's read of it, and between that read and the next write of the place: a wave's
// LDS accesses are carried out in the order they are issued, so nothing has to be waited for, but the compiler, which sees one
// lane, may not move them past each other.
__device__ __forceinline__ void wave_sees_lds() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }

// Where a request's keys lie.
struct Walk {
  typedef const __attribute__((address_space(4))) int32_t* const_i32_ptr;
  const_i32_ptr ids;
  int last_page;
  int L;
  int64_t page_stride;
  __device__ __forceinline__ Walk(const AttnArgs& a, const Work& work, int page_head_bytes) {
    L = work.prefix + work.chunk;
    last_page = (L - 1) / kPageTokens;
    ids = (const_i32_ptr)(a.block_tables + (int64_t)work.req * a.max_pages);
    page_stride = (int64_t)a.Hkv * page_head_bytes;
  }
  // the table is never read past the request's pages
  template <int PAGES>
  __device__ __forceinline__ void pages_of(int block, int (&pid)[PAGES]) const {
#pragma unroll
    for (int h = 0; h < PAGES; ++h) {
      const int lp = block * PAGES + h;
      pid[h] = ids[lp < last_page ? lp : last_page];
    }
  }
};

// 32-key blocks [first, end) of the keys up to token tok_last that are the workgroup's: all of them, or its piece's key tiles
__device__ __forceinline__ void blocks_of(const Work& work, int tok_last, int* first, int* end) {
  constexpr int kBlocks = kTileKeys / 32;
  const int keys = work.prefix + tok_last + 1, all = (keys + 31) / 32;
  int lo, hi;
  piece_tiles((keys + kTileKeys - 1) / kTileKeys, work.piece, work.pieces, &lo, &hi);
  *first = lo * kBlocks;
  *end = hi * kBlocks < all ? hi * kBlocks : all;
}

// A wave's K block on its way to fragments: loaded as it lies (a quarter of a wave takes 256 contiguous bytes; lanes that load
// their own fragments read 16 rows at once), turned in the wave's own corner of LDS.  Rows dense, 16-byte granules swizzled
// so that neither side has bank conflicts.
template <int ROW_BYTES, int PAGES>
struct StageK {
  static constexpr int kGran = ROW_BYTES / 16, kShift = ROW_BYTES == 256 ? 0 : 1;
  static constexpr int kChunks = kPageTokens * ROW_BYTES / 1024, kSteps = ROW_BYTES / 64;
  static __device__ __forceinline__ int swz(int row) { return (row >> kShift) & (kGran - 1); }
  u32x4 raw[PAGES][kChunks];
  __device__ __forceinline__ void load(const Walk& walk, const char* kbase, const int (&pid)[PAGES]) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int h = 0; h < PAGES; ++h) {
      const char* page = kbase + (int64_t)pid[h] * walk.page_stride;
#pragma unroll
      for (int i = 0; i < kChunks; ++i) raw[h][i] = *reinterpret_cast<const u32x4*>(page + (uint32_t)(lane * 16) + i * 1024);
    }
  }
  __device__ __forceinline__ void put(char* lds) const {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int h = 0; h < PAGES; ++h)
#pragma unroll
      for (int i = 0; i < kChunks; ++i) {
        const int row = i * (1024 / ROW_BYTES) + lane / kGran;
        *reinterpret_cast<u32x4*>(lds + (h * kPageTokens + row) * ROW_BYTES + ((lane % kGran ^ swz(row)) << 4)) = raw[h][i];
      }
  }
  // granule 4 step + lane / 16 of row lane % 16 of page h
  template <typename V>
  static __device__ __forceinline__ V fragment(const char* lds, int h, int step) {
    const int lane = threadIdx.x & 63, g = lane >> 4, j = lane & 15;
    return *reinterpret_cast<const V*>(lds + (h * kPageTokens + j) * ROW_BYTES + (((4 * step + g) ^ swz(j)) << 4));
  }
};

// RT: 16-row tiles of a wave.  Two share every K and V fragment; one where no request has more rows (us, two / one: 64/8 heads,
// P 30000, C 1 149 / 139; P 1023, C 2 10.3 / 8.8; 16/16 heads, P 300, C 16 6.7 / 5.9; head_dim 64, 64/8 heads, P 30000, C 2
// 104 / 85).  250 random batches, one-shot and planned: 34 calls of at most 16 rows are 1.04-1.22
// times as fast, none loses.
template <int D, int RT, int SPLIT>
__device__ __forceinline__ void narrow_bf16(const AttnArgs& a, const Work& work, int share) {
  constexpr int kBlockKeys = 32, kBlockPages = kBlockKeys / kPageTokens;
  constexpr int kRows = 16 * RT, kSteps = D / 32, kVec = D / 16 / SPLIT, kRowB = D * 2, kPageHeadB = kPageTokens * kRowB;
  typedef Narrow<kRows, D, SPLIT, kBlockKeys, __bf16> N;
  typedef uint32_t vvec __attribute__((ext_vector_type(kVec / 2)));
  __shared__ __attribute__((aligned(256))) typename N::Shared sh;

  const int lane = threadIdx.x & 63, g = lane >> 4, j = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  char* const k_lds = sh.corner[wave];
  const int G = a.G, n_rows = work.chunk * G;
  const Walk walk(a, work, kPageHeadB);

  int tok[RT];
  bf16x8 qf[kSteps][RT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    int row = work.row0 + rt * 16 + j;
    row = row < n_rows ? row : n_rows - 1;                 // rows past the chunk's end compute the last one again
    tok[rt] = row / G;
    const int64_t at = (int64_t)(work.q_off + tok[rt]) * a.Hq + work.kv_head * G + (row - tok[rt] * G);
    const char* qrow = reinterpret_cast<const char*>(a.q) + at * kRowB;
#pragma unroll
    for (int c = 0; c < kSteps; ++c) qf[c][rt] = *reinterpret_cast<const bf16x8*>(qrow + c * 64 + g * 16);
  }
  const int tok_first = work.row0 / G;
  int tok_last = (work.row0 + kRows - 1) / G;
  tok_last = tok_last < work.chunk - 1 ? tok_last : work.chunk - 1;
  int first_block, n_blocks;
  blocks_of(work, tok_last, &first_block, &n_blocks);
  const int seen_by_all = work.prefix + tok_first + 1;

  const char* kbase = reinterpret_cast<const char*>(a.k_pool) + (int64_t)work.kv_head * kPageHeadB;
  const char* vbase = reinterpret_cast<const char*>(a.v_pool) + (int64_t)work.kv_head * kPageHeadB;
  const uint32_t v_lane = (uint32_t)(4 * g * kRowB + share * (kRowB / SPLIT) + j * (kVec * 2));
  StageK<kRowB, kBlockPages> stage;
  vvec vr[8];                                              // 4 page + r: key 4 g + r of that page
  auto load_v = [&](const int (&pid)[kBlockPages]) __attribute__((always_inline)) {
#pragma unroll
    for (int h = 0; h < kBlockPages; ++h) {
      const char* page = vbase + (int64_t)pid[h] * walk.page_stride;
#pragma unroll
      for (int r = 0; r < 4; ++r) vr[4 * h + r] = *reinterpret_cast<const vvec*>(page + v_lane + r * kRowB);
    }
  };

  f32x4 o[kVec][RT], l_acc[RT];
  float m_run[RT];
  bf16x8 ones;
#pragma unroll
  for (int e = 0; e < 8; ++e) ones[e] = (__bf16)1.0f;
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    m_run[rt] = -INFINITY;
    l_acc[rt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int e = 0; e < kVec; ++e) o[e][rt] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  const float c = a.scale_log2e;

  // Loads are never skipped: behind a branch the compiler could not count those in flight and would wait for all of them.
  // What the last turn loads (its own block again) nobody uses.
  auto next_after = [&](int b) __attribute__((always_inline)) { return b + kWaves < n_blocks ? b + kWaves : b; };
  int pid[kBlockPages];
  int block = first_block + wave;
  if (block < n_blocks) {
    walk.pages_of(block, pid);
    stage.load(walk, kbase, pid);
    load_v(pid);
    walk.pages_of(next_after(block), pid);
  }
  for (; block < n_blocks; block += kWaves) {
    stage.put(k_lds);
    stage.load(walk, kbase, pid);
    wave_sees_lds();
    __builtin_amdgcn_sched_barrier(0);
    f32x4 s[RT][kBlockPages];                               // keys 16 kt + 4 g + r of the block
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int kt = 0; kt < kBlockPages; ++kt) s[rt][kt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int st = 0; st < kSteps; ++st)
#pragma unroll
      for (int kt = 0; kt < kBlockPages; ++kt) {
        const bf16x8 kf = stage.template fragment<bf16x8>(k_lds, kt, st);
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) s[rt][kt] = mma(kf, qf[st][rt], s[rt][kt]);
      }
    if ((block + 1) * kBlockKeys > seen_by_all) {
      asm volatile("");                                    // (a branch, not selects on every block's path)
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        const int lim = work.prefix + tok[rt] - block * kBlockKeys - 4 * g;
#pragma unroll
        for (int kt = 0; kt < kBlockPages; ++kt)
#pragma unroll
          for (int r = 0; r < 4; ++r) s[rt][kt][r] = 16 * kt + r <= lim ? s[rt][kt][r] : -INFINITY;
      }
    }
    if ((block + 1) * kBlockKeys > walk.L) {               // slots at or past the request's length may hold anything
      asm volatile("");
#pragma unroll
      for (int q = 0; q < 8; ++q)
        if (block * kBlockKeys + (q >> 2) * 16 + 4 * g + (q & 3) >= walk.L) vr[q] = vvec{};
    }
    float mx[RT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      mx[rt] = max_over_groups(max8(s[rt][0], s[rt][1])) * c;
    }
    if (__builtin_amdgcn_ballot_w64(mx[0] > m_run[0] + kRescaleSlack || mx[RT - 1] > m_run[RT - 1] + kRescaleSlack) != 0) {
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        const float m_new = fmaxf(m_run[rt], mx[rt]);
        const float alpha = m_new == -INFINITY ? 1.f : __builtin_amdgcn_exp2f(m_run[rt] - m_new);
        m_run[rt] = m_new;
        l_acc[rt] *= alpha;
#pragma unroll
        for (int e = 0; e < kVec; ++e) o[e][rt] *= alpha;
      }
    }
    u32x4 p[RT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      const float ref = fmaxf(m_run[rt], kNoKeyYet);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        typedef float f32x2 __attribute__((ext_vector_type(2)));
        typedef __attribute__((__vector_size__(4))) __bf16 bf16x2;
        f32x2 pp;
#pragma unroll
        for (int e = 0; e < 2; ++e)
          pp[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[rt][k >> 1][(k & 1) * 2 + e], c, -ref));
        p[rt][k] = __builtin_bit_cast(uint32_t, __builtin_convertvector(pp, bf16x2));
      }
      l_acc[rt] = mma(ones, __builtin_bit_cast(bf16x8, p[rt]), l_acc[rt]);
    }
#pragma unroll
    for (int e = 0; e < kVec; ++e) {
      u32x4 w;
#pragma unroll
      for (int k = 0; k < 4; ++k)
        w[k] = __builtin_amdgcn_perm(vr[2 * k + 1][e >> 1], vr[2 * k][e >> 1], (e & 1) ? 0x07060302u : 0x05040100u);
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
        o[e][rt] = mma(__builtin_bit_cast(bf16x8, w), __builtin_bit_cast(bf16x8, p[rt]), o[e][rt]);
    }
    load_v(pid);
    walk.pages_of(next_after(next_after(block)), pid);
    wave_sees_lds();
    __builtin_amdgcn_sched_barrier(0);
  }

  // column kVec (4 g + r) + e of the share, row 16 rt + j
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    const int row = rt * 16 + j;
    constexpr int kStore = kVec < 4 ? kVec : 4;
    typedef float fvec __attribute__((ext_vector_type(kStore)));
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int e = 0; e < kVec; e += kStore) {
        fvec v;
#pragma unroll
        for (int i = 0; i < kStore; ++i) v[i] = o[e + i][rt][r];
        *reinterpret_cast<fvec*>(sh.o(wave, row) + kVec * (4 * g + r) + e) = v;
      }
    if (g == 0) {
      sh.m[wave][row] = m_run[rt];
      sh.l[wave][row] = l_acc[rt][0];
    }
  }
  __syncthreads();
  N::finish(sh, a, work, share, n_rows);
}

template <int SPLIT>
__device__ __forceinline__ void narrow_f32(const AttnArgs& a, const Work& work, int share) {
  constexpr int kRows = 16, D = 64, kVec = D / 16 / SPLIT, kBlockKeys = 32, kBlockPages = kBlockKeys / kPageTokens;
  typedef Narrow<kRows, D, SPLIT, kBlockKeys, float> N;
  typedef float fvec __attribute__((ext_vector_type(kVec)));
  __shared__ __attribute__((aligned(256))) typename N::Shared sh;

  const int lane = threadIdx.x & 63, g = lane >> 4, j = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  char* const k_lds = sh.corner[wave];
  const int G = a.G, n_rows = work.chunk * G;
  const Walk walk(a, work, kPageHeadBytes);

  int row = work.row0 + j;
  row = row < n_rows ? row : n_rows - 1;
  const int tok = row / G;
  f32x4 qf[4];                                             // step (i, e) of the contraction takes column 16 i + 4 g + e
  {
    const int64_t at = (int64_t)(work.q_off + tok) * a.Hq + work.kv_head * G + (row - tok * G);
    const char* qrow = reinterpret_cast<const char*>(a.q) + at * kRowBytes;
#pragma unroll
    for (int i = 0; i < 4; ++i) qf[i] = *reinterpret_cast<const f32x4*>(qrow + i * 64 + g * 16);
  }
  const int tok_first = work.row0 / G;
  int tok_last = (work.row0 + kRows - 1) / G;
  tok_last = tok_last < work.chunk - 1 ? tok_last : work.chunk - 1;
  int first_block, n_blocks;
  blocks_of(work, tok_last, &first_block, &n_blocks);
  const int seen_by_all = work.prefix + tok_first + 1;

  const char* kbase = reinterpret_cast<const char*>(a.k_pool) + (int64_t)work.kv_head * kPageHeadBytes;
  const char* vbase = reinterpret_cast<const char*>(a.v_pool) + (int64_t)work.kv_head * kPageHeadBytes;
  const uint32_t v_lane = (uint32_t)(4 * g * kRowBytes + share * (kRowBytes / SPLIT) + j * (kVec * 4));
  StageK<kRowBytes, kBlockPages> stage;
  fvec vr[8];
  auto load_v = [&](const int (&pid)[kBlockPages]) __attribute__((always_inline)) {
#pragma unroll
    for (int h = 0; h < kBlockPages; ++h) {
      const char* page = vbase + (int64_t)pid[h] * walk.page_stride;
#pragma unroll
      for (int r = 0; r < 4; ++r) vr[4 * h + r] = *reinterpret_cast<const fvec*>(page + v_lane + r * kRowBytes);
    }
  };

  f32x4 o[kVec];
#pragma unroll
  for (int e = 0; e < kVec; ++e) o[e] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m_run = -INFINITY, l_run = 0.f;                    // (l_run: this lane group's keys)
  const float c = a.scale_log2e;

  // Loads are never skipped: behind a branch the compiler could not count those in flight and would wait for all of them.
  // What the last turn loads (its own block again) nobody uses.
  auto next_after = [&](int b) __attribute__((always_inline)) { return b + kWaves < n_blocks ? b + kWaves : b; };
  int pid[kBlockPages];
  int block = first_block + wave;
  if (block < n_blocks) {
    walk.pages_of(block, pid);
    stage.load(walk, kbase, pid);
    load_v(pid);
    walk.pages_of(next_after(block), pid);
  }
  for (; block < n_blocks; block += kWaves) {
    stage.put(k_lds);
    stage.load(walk, kbase, pid);
    wave_sees_lds();
    __builtin_amdgcn_sched_barrier(0);
    f32x4 s[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const f32x4 k0 = stage.template fragment<f32x4>(k_lds, 0, i), k1 = stage.template fragment<f32x4>(k_lds, 1, i);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        s[0] = mma(k0[e], qf[i][e], s[0]);
        s[1] = mma(k1[e], qf[i][e], s[1]);
      }
    }
    if ((block + 1) * kBlockKeys > seen_by_all) {
      asm volatile("");
      const int lim = work.prefix + tok - block * kBlockKeys - 4 * g;
#pragma unroll
      for (int kt = 0; kt < 2; ++kt)
#pragma unroll
        for (int r = 0; r < 4; ++r) s[kt][r] = 16 * kt + r <= lim ? s[kt][r] : -INFINITY;
    }
    if ((block + 1) * kBlockKeys > walk.L) {
      asm volatile("");
#pragma unroll
      for (int q = 0; q < 8; ++q)
        if (block * kBlockKeys + (q >> 2) * 16 + 4 * g + (q & 3) >= walk.L) vr[q] = fvec{};
    }
    const float mx = max_over_groups(max8(s[0], s[1])) * c;
    if (__builtin_amdgcn_ballot_w64(mx > m_run + kRescaleSlack) != 0) {
      const float m_new = fmaxf(m_run, mx);
      const float alpha = m_new == -INFINITY ? 1.f : __builtin_amdgcn_exp2f(m_run - m_new);
      m_run = m_new;
      l_run *= alpha;
#pragma unroll
      for (int e = 0; e < kVec; ++e) o[e] *= alpha;
    }
    const float ref = fmaxf(m_run, kNoKeyYet);
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        s[kt][r] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[kt][r], c, -ref));
        l_run += s[kt][r];
      }
#pragma unroll
    for (int q = 0; q < 8; ++q)
#pragma unroll
      for (int e = 0; e < kVec; ++e) o[e] = mma(vr[q][e], s[q >> 2][q & 3], o[e]);
    load_v(pid);
    walk.pages_of(next_after(next_after(block)), pid);
    wave_sees_lds();
    __builtin_amdgcn_sched_barrier(0);
  }

  l_run += __shfl_xor(l_run, 16, 64);
  l_run = sum_with_other_half(l_run);
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    fvec v;
#pragma unroll
    for (int e = 0; e < kVec; ++e) v[e] = o[e][r];
    *reinterpret_cast<fvec*>(sh.o(wave, j) + kVec * (4 * g + r)) = v;
  }
  if (g == 0) {
    sh.m[wave][j] = m_run;
    sh.l[wave][j] = l_run;
  }
  __syncthreads();
  N::finish(sh, a, work, share, n_rows);
}

// BF16_D: head_dim of the bf16 forms, 0: fp32
template <int BF16_D, int ROWS, int SPLIT>
__device__ __forceinline__ void narrow_body(const AttnArgs& a, const Work& work, int share) {
  if constexpr (BF16_D == 0) narrow_f32<SPLIT>(a, work, share);
  else narrow_bf16<BF16_D, ROWS / 16, SPLIT>(a, work, share);
}

template <int BF16_D, int ROWS>
__global__ __launch_bounds__(kWaves * 64) void attn_narrow_classes_kernel(const AttnArgs a, const AttnClasses t) {
  narrow_body<BF16_D, ROWS, 1>(a, work_of<ROWS>(t, blockIdx.x, a.Hkv, a.G), 0);
}
// workgroups n_items k .. take the k-th share of the columns
template <int BF16_D, int ROWS, int SPLIT>
__global__ __launch_bounds__(kWaves * 64) void attn_narrow_shared_classes_kernel(const AttnArgs a, const AttnClasses t) {
  const int share = (int)blockIdx.x / a.n_items;
  narrow_body<BF16_D, ROWS, SPLIT>(a, work_of<ROWS>(t, (int)blockIdx.x - share * a.n_items, a.Hkv, a.G), share);
}

// workgroups n_items k .. take the (k / SPLIT)-th ROWS rows of the items, and of their columns share k % SPLIT
template <int BF16_D, int ROWS, int SPLIT>
__device__ __forceinline__ void narrow_list(const AttnArgs& a) {
  const int part = (int)blockIdx.x / a.n_items;
  const AttnItem item = a.items[(int)blockIdx.x - part * a.n_items];
  const AttnReq rq = a.reqs[item.req];
  const int row0 = item.row0 + part / SPLIT * ROWS;
  if (row0 >= rq.chunk * a.G) return;
  narrow_body<BF16_D, ROWS, SPLIT>(a, Work{item.req, item.kv_head, row0, rq.q_off, rq.prefix, rq.chunk, 0, 1, 0, false}, part % SPLIT);
}
template <int BF16_D, int ROWS>
__global__ __launch_bounds__(kWaves * 64) void attn_narrow_list_kernel(const AttnArgs a) {
  narrow_list<BF16_D, ROWS, 1>(a);
}
template <int BF16_D, int ROWS, int SPLIT>
__global__ __launch_bounds__(kWaves * 64) void attn_narrow_shared_list_kernel(const AttnArgs a) {
  narrow_list<BF16_D, ROWS, SPLIT>(a);
}

template <int BF16_D, int ROWS, int SPLIT>
void enqueue(const AttnArgs& args, int parts, const AttnClasses* t, hipStream_t stream) {
  if constexpr (SPLIT == 1) {
    if (t != nullptr) attn_narrow_classes_kernel<BF16_D, ROWS><<<args.n_items, kWaves * 64, 0, stream>>>(args, *t);
    else attn_narrow_list_kernel<BF16_D, ROWS><<<args.n_items * parts, kWaves * 64, 0, stream>>>(args);
  } else {
    if (t != nullptr) attn_narrow_shared_classes_kernel<BF16_D, ROWS, SPLIT><<<args.n_items * SPLIT, kWaves * 64, 0, stream>>>(args, *t);
    else attn_narrow_shared_list_kernel<BF16_D, ROWS, SPLIT><<<args.n_items * parts * SPLIT, kWaves * 64, 0, stream>>>(args);
  }
}
// (head_dim 64 in bf16: a quarter of the columns is no sooner than half of them)
template <int BF16_D, int ROWS>
void enqueue(const AttnArgs& args, int parts, int shares, const AttnClasses* t, hipStream_t stream) {
  if (shares == 4 && BF16_D != 64) enqueue<BF16_D, ROWS, BF16_D == 64 ? 2 : 4>(args, parts, t, stream);
  else if (shares > 1) enqueue<BF16_D, ROWS, 2>(args, parts, t, stream);
  else enqueue<BF16_D, ROWS, 1>(args, parts, t, stream);
}

}  // namespace

hipError_t launch_attn_narrow(int dtype, const AttnArgs& args, int rows, int parts, int shares, const AttnClasses* t,
                              hipStream_t stream) {
  (void)hipGetLastError();
  const bool bf16 = dtype == MC_DTYPE_BF16, least = rows == kAttnLeastRows;
  if (!least && !(bf16 && rows == kAttnNarrowRows)) return hipErrorInvalidValue;
  if (dtype == MC_DTYPE_F32 && args.head_dim == 64)
    enqueue<0, kAttnLeastRows>(args, parts, shares, t, stream);
  else if (bf16 && args.head_dim == 128)
    least ? enqueue<128, kAttnLeastRows>(args, parts, shares, t, stream) : enqueue<128, kAttnNarrowRows>(args, parts, shares, t, stream);
  else if (bf16 && args.head_dim == 64)
    least ? enqueue<64, kAttnLeastRows>(args, parts, shares, t, stream) : enqueue<64, kAttnNarrowRows>(args, parts, shares, t, stream);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace mc
