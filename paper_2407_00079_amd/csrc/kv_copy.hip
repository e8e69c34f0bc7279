// Layer-wise KV page movement (paper Section 5.2: per-layer KVCache load before
// attention, store after it): gather scattered pages into a contiguous per-layer
// buffer (pack) and scatter such a buffer into scattered pages (unpack).
//
// Pure HBM traffic, no arithmetic: every byte is read once and written once with
// 128-bit nontemporal accesses.  One workgroup moves one 8 KiB slice of one page;
// its page id is a single uniform (scalar) load.  Many small workgroups (16 Ki of
// them for a 32 KiB-page layer) measured best here: slices of 4..32 KiB, 64..1024
// threads, and persistent grids all land within a few percent of each other, at
// the rate the HBM sustains for a read+write mix.
//
// Also here, all of them byte movers or integer scans over page id lists: the ranking of a page
// list by pool address (so that the scattered side of a copy can walk the pool front to back),
// the range check of an id list, and the append of a chunk's new K/V rows into their page slots.
#include "mc_internal.h"

namespace mc {
namespace {

constexpr int kThreads = 512;
constexpr int kUnroll = 1;                        // 16-byte vectors per thread
constexpr int kSliceVecs = kThreads * kUnroll;    // 8 KiB per workgroup
static_assert(kSliceVecs == kKvCopySliceVecs, "the host sizes the copy grid with kKvCopySliceVecs");

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

template <bool kPack>
__global__ __launch_bounds__(kThreads) void kv_copy_kernel(const u32x4* __restrict__ k_src,
                                                           const u32x4* __restrict__ v_src,
                                                           u32x4* __restrict__ k_dst,
                                                           u32x4* __restrict__ v_dst,
                                                           const int32_t* __restrict__ page_ids,
                                                           const int32_t* __restrict__ order,
                                                           int64_t page_vecs, int slices_per_page) {
  const int turn = blockIdx.x / slices_per_page;
  const int slice = blockIdx.x - turn * slices_per_page;
  // Workgroups start in blockIdx order.  With `order` (list positions by ascending pool page) the
  // scattered side of the copy walks the pool in address order, which the HBM takes better
  // than a random walk (unpack: 5.6 -> 6.1 TB/s on a 32 KiB-page layer); what is copied where is
  // the same either way.
  const int page = order != nullptr ? order[turn] : turn;
  const int64_t pool_page = page_ids[page];
  const u32x4* src = blockIdx.y ? v_src : k_src;
  u32x4* dst = blockIdx.y ? v_dst : k_dst;
  // pack: pool page -> list position; unpack: list position -> pool page
  src += (kPack ? pool_page : (int64_t)page) * page_vecs;
  dst += (kPack ? (int64_t)page : pool_page) * page_vecs;

  const int64_t first = (int64_t)slice * kSliceVecs + threadIdx.x;
  u32x4 v[kUnroll];
  if (first + (kUnroll - 1) * kThreads < page_vecs) {
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) v[u] = __builtin_nontemporal_load(src + first + u * kThreads);
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) __builtin_nontemporal_store(v[u], dst + first + u * kThreads);
  } else {
#pragma unroll
    for (int u = 0; u < kUnroll; ++u)
      if (first + u * kThreads < page_vecs) v[u] = __builtin_nontemporal_load(src + first + u * kThreads);
#pragma unroll
    for (int u = 0; u < kUnroll; ++u)
      if (first + u * kThreads < page_vecs) __builtin_nontemporal_store(v[u], dst + first + u * kThreads);
  }
}

// A layer's load or store in one launch, where it is small: the kernel reads or writes pinned host memory itself and leaves the
// packed form in the staging buffers on the way.  What bounds it: the host link (55 GB/s).  The copy engine's way is two copies and
// a kernel, each waiting for the one before through a signal (20-130 us of an idle link between them), and copies of several
// streams wait for each other where they share an engine.  Four layers of K and V each way on two streams, three such pairs of
// streams in turn, us by the copy engine / so: 64 KiB a copy 178-203 / 157, 512 KiB 438 / 178, 1 MiB 656 / 321, 2 MiB 940 / 596;
// 12.6 MB in by the engine and 1.67 MB out 2837 / 2204.
// Few workgroups, small enough to run beside attention's on a compute unit: 16 keep 256 KiB of reads in flight, and 8 write as
// fast as the link takes it while fewer of attention's wait behind them.  A step of 231 us of attention a layer (64/8 heads, P 8192,
// C 1024) that stores 2 MiB of K and of V 376 by the engine, with 64 workgroups 304, 16 296, 8 292; one of 1010 us of attention
// 1047, 1079, 1060, 1057 (loads make no difference).  So no stores beyond 2 MiB: the engine disturbs a long attention less.  Loads
// stop there too, without having been weighed by themselves.
constexpr int kHostThreads = 256, kHostPer = 4, kHostLoadGrid = 16, kHostStoreGrid = 8;
static_assert(kHostThreads * 16 == kHostSliceBytes, "a workgroup moves a slice at a time");
template <bool kLoad>
__global__ __launch_bounds__(kHostThreads) void kv_host_kernel(u32x4* k_host, u32x4* v_host, u32x4* k_stage, u32x4* v_stage,
                                                               u32x4* k_pool, u32x4* v_pool,
                                                               const int32_t* __restrict__ page_ids, int page_vecs,
                                                               int slices_per_page, int slices) {
  for (int base = blockIdx.x; base < 2 * slices; base += kHostPer * gridDim.x) {
    u32x4 v[kHostPer];
    // slice `at` of K, then of V: page, vector of the page, and whether the thread has one
    auto each = [&](auto&& move) __attribute__((always_inline)) {
#pragma unroll
      for (int u = 0; u < kHostPer; ++u) {
        const int at = base + u * (int)gridDim.x;
        if (at >= 2 * slices) break;
        const bool second = at >= slices;
        const int rest = second ? at - slices : at, page = rest / slices_per_page;
        const int vec = (rest - page * slices_per_page) * kHostThreads + (int)threadIdx.x;
        if (vec < page_vecs) move(v[u], second, (int64_t)page * page_vecs + vec, (int64_t)page_ids[page] * page_vecs + vec);
      }
    };
    each([&](u32x4& x, bool second, int64_t packed, int64_t paged) __attribute__((always_inline)) {
      x = kLoad ? (second ? v_host : k_host)[packed] : (second ? v_pool : k_pool)[paged];
    });
    each([&](u32x4& x, bool second, int64_t packed, int64_t paged) __attribute__((always_inline)) {
      (second ? v_stage : k_stage)[packed] = x;
      if (kLoad) (second ? v_pool : k_pool)[paged] = x;
      else (second ? v_host : k_host)[packed] = x;
    });
  }
}

// order[r] = the list position whose pool page is the r-th smallest (ties: lower position first),
// i.e. the rank of the 64-bit key (page id, list position).  Rank by counting, the ids staged
// through LDS in chunks: O(n^2) compares, meant to be run once per request - the list is the same
// for every layer.  LANES threads share a position, each counting every LANES-th group of four
// keys, so that short lists fill the chip too (2048 ids: 8 workgroups and 26 us with one thread a
// position, 128 and 5 us with 16).  Slots past the end of the list hold the largest id at
// positions behind all others and count nothing.
constexpr int kOrderChunk = 1024;
template <int LANES>
__global__ __launch_bounds__(256) void kv_page_order_kernel(const int32_t* __restrict__ page_ids, int64_t n,
                                                            int32_t* __restrict__ order) {
  __shared__ u32x4 chunk[kOrderChunk / 4];
  const int part = threadIdx.x % LANES;
  const int64_t i = (int64_t)blockIdx.x * (256 / LANES) + threadIdx.x / LANES;
  // ids are not negative and positions stay below 2^20: (id << 32) | position orders as the pair does
  const uint64_t mine = i < n ? ((uint64_t)(uint32_t)page_ids[i] << 32) | (uint64_t)i : 0;
  int rank = 0;
  for (int64_t base = 0; base < n; base += kOrderChunk) {
    __syncthreads();
    const int64_t at = base + threadIdx.x * 4;
    u32x4 ids;
#pragma unroll
    for (int e = 0; e < 4; ++e) ids[e] = at + e < n ? (uint32_t)page_ids[at + e] : ~0u;
    chunk[threadIdx.x] = ids;
    __syncthreads();
#pragma unroll 8
    for (int t = part; t < kOrderChunk / 4; t += LANES) {
      const u32x4 o = chunk[t];
      const uint32_t pos = (uint32_t)base + 4 * t;
#pragma unroll
      for (int e = 0; e < 4; ++e) rank += (((uint64_t)o[e] << 32) | (pos + e)) < mine;
    }
  }
#pragma unroll
  for (int d = LANES / 2; d >= 1; d >>= 1) rank += __shfl_xor(rank, d, 64);
  if (i < n && part == 0) order[rank] = (int32_t)i;
}

// Range check of a page id list (debugging aid): a one-thread kernel resets the report, then every
// wave counts its out-of-range ids and adds them with one atomic; the first position by atomicMin.
__global__ void kv_check_reset_kernel(int32_t* __restrict__ report, int32_t n) {
  report[0] = 0;
  report[1] = n;
}

__global__ __launch_bounds__(256) void kv_check_page_ids_kernel(const int32_t* __restrict__ page_ids, int64_t n,
                                                                int64_t num_pages, int32_t* __restrict__ report) {
  int count = 0;
  int64_t first = n;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    const int64_t id = page_ids[i];
    if (id < 0 || id >= num_pages) {
      ++count;
      first = i < first ? i : first;
    }
  }
  if (__builtin_amdgcn_ballot_w64(count != 0) == 0) return;    // the usual case: nothing to report
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) {
    count += __shfl_xor(count, d, 64);
    const int other = __shfl_xor((int)first, d, 64);
    first = other < first ? other : first;
  }
  if ((threadIdx.x & 63) == 0) {
    atomicAdd(report, count);
    atomicMin(report + 1, (int)first);
  }
}

// Append (paper Section 3 step 2: the chunk's new KVCache is kept in the request's pages):
// one thread moves one 16-byte granule of one (token, KV head) row of K and of V; a row has 1 << gran_shift granules
// (256 bytes for bf16 head_dim 128 and fp32 head_dim 64, 128 bytes for bf16 head_dim 64).  The request of a token is the
// last one that starts at or before it: requests without new tokens share their start with the next one, and the last of
// such a run is the one that owns the token.
__device__ __forceinline__ int owner_of(const AttnReq* reqs, int batch, int32_t tok) {
  int lo = 0, hi = batch - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (reqs[mid].q_off <= tok) lo = mid; else hi = mid - 1;
  }
  return lo;
}
// a table in the kernel argument: each lane looks at one request for the wave's first token, and the threads whose token
// lies in a later request (few waves have any) walk on from there
__device__ __forceinline__ int owner_of(const AttnReqTable& t, int batch, int32_t tok) {
  const int lane = threadIdx.x & 63;
  const int32_t first = __builtin_amdgcn_readfirstlane(tok);
  int r = __popcll(__builtin_amdgcn_ballot_w64(lane < batch && t.r[lane].q_off <= first)) - 1;
  while (r + 1 < batch && t.r[r + 1].q_off <= tok) ++r;
  return r;
}
__device__ __forceinline__ AttnReq req_at(const AttnReq* reqs, int i) { return reqs[i]; }
__device__ __forceinline__ AttnReq req_at(const AttnReqTable& t, int i) { return t.r[i]; }

template <typename Reqs>      // const AttnReq* or AttnReqTable
__global__ __launch_bounds__(256) void kv_append_kernel(const u32x4* __restrict__ k_new, const u32x4* __restrict__ v_new,
                                                        u32x4* __restrict__ k_pool, u32x4* __restrict__ v_pool,
                                                        const int32_t* __restrict__ block_tables, int32_t max_pages,
                                                        const Reqs reqs, int32_t batch, int64_t total_vecs, int32_t Hkv,
                                                        int32_t gran_shift) {
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  // threads past the end stay for the search (it looks at one request per lane) with the last granule's token
  const int64_t at = idx < total_vecs ? idx : total_vecs - 1;
  const int gran = (int)(at & ((1 << gran_shift) - 1));
  const int64_t row = at >> gran_shift;         // (token, head)
  const int g = (int)(row % Hkv);
  const int32_t tok = (int32_t)(row / Hkv);
  const int owner = owner_of(reqs, batch, tok);
  if (idx >= total_vecs) return;
  const AttnReq rq = req_at(reqs, owner);
  const int32_t pos = rq.prefix + (tok - rq.q_off);
  const int64_t page = block_tables[(int64_t)owner * max_pages + (pos >> 4)];
  const int64_t dst = ((((page * Hkv + g) << 4) + (pos & 15)) << gran_shift) + gran;
  k_pool[dst] = k_new[idx];
  v_pool[dst] = v_new[idx];
}

}  // namespace

hipError_t launch_kv_page_order(const int32_t* page_ids, int64_t n, int32_t* order, hipStream_t stream) {
  (void)hipGetLastError();
  // as many threads a position as it takes to fill 256 compute units; every workgroup stages the whole list, so not more
  auto blocks = [&](int per) { return (unsigned)((n + per - 1) / per); };
  if (n <= 8192) kv_page_order_kernel<16><<<blocks(16), 256, 0, stream>>>(page_ids, n, order);
  else if (n <= 32768) kv_page_order_kernel<4><<<blocks(64), 256, 0, stream>>>(page_ids, n, order);
  else kv_page_order_kernel<1><<<blocks(256), 256, 0, stream>>>(page_ids, n, order);
  return hipGetLastError();
}

hipError_t launch_kv_check_page_ids(const int32_t* page_ids, int64_t n, int64_t num_pages, int32_t* report,
                                    hipStream_t stream) {
  (void)hipGetLastError();
  kv_check_reset_kernel<<<1, 1, 0, stream>>>(report, (int32_t)n);
  const int64_t blocks = (n + 255) / 256;
  kv_check_page_ids_kernel<<<(unsigned)(blocks < 4096 ? blocks : 4096), 256, 0, stream>>>(page_ids, n, num_pages, report);
  return hipGetLastError();
}

hipError_t launch_kv_append(const void* k_new, const void* v_new, void* k_pool, void* v_pool,
                            const int32_t* block_tables, int32_t max_pages, const AttnReq* reqs, const AttnReqTable* arg,
                            int32_t batch, int64_t total_new, int32_t Hkv, int32_t row_bytes, hipStream_t stream) {
  const int32_t gran_shift = row_bytes == 256 ? 4 : 3;      // 256- or 128-byte rows
  const int64_t total_vecs = (total_new * Hkv) << gran_shift;
  const unsigned blocks = (unsigned)((total_vecs + 255) / 256);
  (void)hipGetLastError();
  if (arg != nullptr)
    kv_append_kernel<AttnReqTable><<<blocks, 256, 0, stream>>>(
        (const u32x4*)k_new, (const u32x4*)v_new, (u32x4*)k_pool, (u32x4*)v_pool, block_tables, max_pages, *arg, batch,
        total_vecs, Hkv, gran_shift);
  else
    kv_append_kernel<const AttnReq*><<<blocks, 256, 0, stream>>>(
        (const u32x4*)k_new, (const u32x4*)v_new, (u32x4*)k_pool, (u32x4*)v_pool, block_tables, max_pages, reqs, batch,
        total_vecs, Hkv, gran_shift);
  return hipGetLastError();
}

hipError_t launch_kv_host(bool load, void* k_host, void* v_host, void* k_stage, void* v_stage, void* k_pool, void* v_pool,
                          const int32_t* page_ids, int64_t n, int64_t page_bytes, hipStream_t stream) {
  const int per_page = (int)((page_bytes + kHostSliceBytes - 1) / kHostSliceBytes), slices = (int)n * per_page;
  const int most = load ? kHostLoadGrid : kHostStoreGrid;
  const unsigned grid = (unsigned)(2 * slices < most ? 2 * slices : most);
  auto kernel = load ? kv_host_kernel<true> : kv_host_kernel<false>;
  (void)hipGetLastError();
  kernel<<<grid, kHostThreads, 0, stream>>>((u32x4*)k_host, (u32x4*)v_host, (u32x4*)k_stage, (u32x4*)v_stage, (u32x4*)k_pool,
                                            (u32x4*)v_pool, page_ids, (int)(page_bytes / 16), per_page, slices);
  return hipGetLastError();
}

hipError_t launch_kv_copy(bool pack, const void* k_src, const void* v_src, void* k_dst, void* v_dst,
                          const int32_t* page_ids, const int32_t* order, int64_t n, int64_t page_bytes,
                          hipStream_t stream) {
  const int64_t page_vecs = page_bytes / 16;
  const int slices = (int)((page_vecs + kSliceVecs - 1) / kSliceVecs);
  dim3 grid((unsigned)(n * slices), 2, 1);
  (void)hipGetLastError();   // drop any stale error of earlier, unrelated runtime calls
  if (pack)
    kv_copy_kernel<true><<<grid, kThreads, 0, stream>>>((const u32x4*)k_src, (const u32x4*)v_src, (u32x4*)k_dst,
                                                        (u32x4*)v_dst, page_ids, order, page_vecs, slices);
  else
    kv_copy_kernel<false><<<grid, kThreads, 0, stream>>>((const u32x4*)k_src, (const u32x4*)v_src, (u32x4*)k_dst,
                                                         (u32x4*)v_dst, page_ids, order, page_vecs, slices);
  return hipGetLastError();
}

}  // namespace mc
