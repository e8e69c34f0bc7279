// Prefix block keys and longest prefix match for gfx950 (paper Algorithm 1: PrefixHash and
// FindBestPrefixMatch; Figure "KVCache pool": a block's hash value is determined by its own hash
// and by its prefix).  The paper fixes the block size (512 tokens), not the hash; the one used
// here is stated in include/mc.h.  Integer work, bit-exact against the CPU oracle.
//
//   A block's digest is one wave's work (64 partial sums of position-salted mixes, added across the wave) and blocks are
//   independent; the chain that turns a request's digests into keys is sequential, one mix per block.
//   short kernel   requests of few blocks, one workgroup each: digests into LDS, then one wave chains them.
//   stage kernel   longer ones: digests of one range of blocks (four per workgroup) beside the chain of another range
//                  (one wave per request).
//   pour kernel    a queue of them: a workgroup per request chains its first blocks while it digests the later ones.
//   match kernel   one workgroup per (instance, request): thread t looks keys t, t + 256, ... up
//                  in the instance's ascending key array; the smallest index that misses is the
//                  prefix length.
//   best kernel    sixteen lanes per request scan its row of prefix lengths.
//   small match    both of them for requests of few (key, instance) pairs, one workgroup each.
#include "mc_internal.h"

namespace mc {
namespace {

__device__ __forceinline__ uint64_t mix64(uint64_t x) {
  x += 0x9E3779B97F4A7C15ull;
  x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
  x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
  return x ^ (x >> 31);
}

// offset tables in device memory; OffsetTables (same member names) is the form that travels with the launch
struct TablePtrs {
  const int64_t* __restrict__ a;
  const int64_t* __restrict__ b;
};

// Digest of a block of nb tokens, by a whole wave (every lane gets it).  Bound by the vector ALU: about 26 instructions
// per token and lane, six of them 32-bit multiplies at a quarter of the rate (16384 blocks of 512 tokens: 12 us).
__device__ __forceinline__ uint64_t digest_of(const int32_t* __restrict__ t, int nb, int lane) {
  uint64_t sum = 0;
  int j = lane;
  for (; j + 7 * 64 < nb; j += 8 * 64) {                  // eight loads in flight per lane
    int32_t v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = t[j + 64 * u];
#pragma unroll
    for (int u = 0; u < 8; ++u) sum += mix64((uint64_t)(uint32_t)v[u] + ((uint64_t)(j + 64 * u) << 32));
  }
  for (; j < nb; j += 64) sum += mix64((uint64_t)(uint32_t)t[j] + ((uint64_t)j << 32));
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) {
    const uint32_t lo = __shfl_xor((uint32_t)sum, d, 64), hi = __shfl_xor((uint32_t)(sum >> 32), d, 64);
    sum += ((uint64_t)hi << 32) | lo;
  }
  return mix64(sum + (uint64_t)nb);
}

constexpr uint64_t kFirstSalt = 0x243F6A8885A308D3ull;
__device__ __forceinline__ uint64_t salt_after(uint64_t key) { return ((key << 23) | (key >> 41)) * 0x9E3779B97F4A7C15ull; }

// A link of the chain with the block's digest in lane LANE, whose key goes to the same lane of (lo, hi).  (A lane known at
// compile time is an immediate for both lane moves; v_writelane has no builtin.)
template <int LANE>
__device__ __forceinline__ void chain_link(uint64_t digest, uint64_t& salt, uint32_t& lo, uint32_t& hi) {
  const uint32_t dl = __builtin_amdgcn_readlane((uint32_t)digest, LANE);
  const uint32_t dh = __builtin_amdgcn_readlane((uint32_t)(digest >> 32), LANE);
  const uint64_t key = mix64((((uint64_t)dh << 32) | dl) ^ salt);
  salt = salt_after(key);
  asm("v_writelane_b32 %0, %1, %2" : "+v"(lo) : "s"((uint32_t)key), "n"(LANE));
  asm("v_writelane_b32 %0, %1, %2" : "+v"(hi) : "s"((uint32_t)(key >> 32)), "n"(LANE));
}
template <int LANE>
__device__ __forceinline__ void chain_four(uint64_t digest, uint64_t& salt, uint32_t& lo, uint32_t& hi) {
  chain_link<LANE>(digest, salt, lo, hi);
  chain_link<LANE + 1>(digest, salt, lo, hi);
  chain_link<LANE + 2>(digest, salt, lo, hi);
  chain_link<LANE + 3>(digest, salt, lo, hi);
}

__device__ __forceinline__ int64_t uniform64(int64_t x) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)x), hi = __builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)x >> 32));
  return (int64_t)(((uint64_t)hi << 32) | lo);
}

// Blocks [lo, hi) of a request from digests in `from` to keys in `to` (the same array, or LDS and the keys), by one wave,
// 16 blocks a turn.  Bound by the issue of one wave's scalar instructions, about 6 cycles each whatever they are, so a
// link is nothing but the hash: no first-block case, no lane compare, no counter
// (34 instructions, 97 ns; 47 and 118 ns with them: 256 links 30 -> 25 us).
__device__ __forceinline__ void chain_range(const uint64_t* from, uint64_t* to, int64_t lo, int64_t hi, uint64_t& salt, int lane) {
  uint64_t ahead = lane < 16 && lo + lane < hi ? from[lo + lane] : 0;
  for (int64_t base = lo; base < hi; base += 16) {
    const uint64_t digest = ahead;
    const int64_t i = base + lane;
    ahead = lane < 16 && i + 16 < hi ? from[i + 16] : 0;  // in flight while these are chained
    uint32_t kl = 0, kh = 0;
    chain_four<0>(digest, salt, kl, kh);                  // (links past the end lead nowhere: nothing follows them)
    if (base + 4 < hi) chain_four<4>(digest, salt, kl, kh);
    if (base + 8 < hi) chain_four<8>(digest, salt, kl, kh);
    if (base + 12 < hi) chain_four<12>(digest, salt, kl, kh);
    if (lane < 16 && i < hi) to[i] = ((uint64_t)kh << 32) | kl;
  }
}

template <typename Tables>     // a: token offsets, b: key offsets
__global__ __launch_bounds__(1024) void prefix_short_kernel(const int32_t* __restrict__ tokens, const Tables off, int batch,
                                                            int block_tokens, uint64_t* __restrict__ keys) {
  __shared__ uint64_t digests[kShortHashBlocks];
  const int lane = threadIdx.x & 63;
  for (int r = blockIdx.x; r < batch; r += gridDim.x) {
    const int64_t k0 = off.b[r], t0 = off.a[r], len = off.a[r + 1] - t0;
    const int nk = (int)(off.b[r + 1] - k0);
    for (int b = threadIdx.x >> 6; b < nk; b += blockDim.x >> 6) {
      const int64_t at = (int64_t)b * block_tokens, left = len - at;
      const uint64_t d = digest_of(tokens + t0 + at, left < block_tokens ? (int)left : block_tokens, lane);
      if (lane == 0) digests[b] = d;
    }
    __syncthreads();
    uint64_t salt = kFirstSalt;
    if (threadIdx.x < 64) chain_range(digests, keys + k0, 0, nk, salt, lane);
    __syncthreads();
  }
}

// A range of blocks [lo, hi); of a request, those of them it has.
struct Blocks {
  int64_t lo, hi;
};

// Requests sit along blockIdx.x.  Row 0 of the grid, where `chains` says so, chains blocks `chain` of its request (their
// digests are complete, and the key before them); the other rows digest blocks `digest`, four per workgroup and turn.
template <typename Tables>
__global__ __launch_bounds__(256) void prefix_stage_kernel(const int32_t* __restrict__ tokens, const Tables off, int batch,
                                                           int block_tokens, const Blocks digest, const Blocks chain,
                                                           const int chains, uint64_t* keys) {
  const int lane = threadIdx.x & 63;
  const int row = (int)blockIdx.y - chains;
  for (int r = blockIdx.x; r < batch; r += gridDim.x) {
    const int64_t k0 = off.b[r], nk = off.b[r + 1] - k0;
    if (row < 0) {
      if (threadIdx.x >= 64) return;
      const int64_t hi = nk < chain.hi ? nk : chain.hi;
      if (chain.lo >= hi) continue;
      uint64_t salt = chain.lo == 0 ? kFirstSalt : salt_after((uint64_t)uniform64((int64_t)keys[k0 + chain.lo - 1]));
      chain_range(keys + k0, keys + k0, chain.lo, hi, salt, lane);
      continue;
    }
    const int64_t t0 = off.a[r], len = off.a[r + 1] - t0;
    const int64_t hi = nk < digest.hi ? nk : digest.hi;
    for (int64_t b = digest.lo + (int64_t)row * 4 + (threadIdx.x >> 6); b < hi; b += (int64_t)(gridDim.y - chains) * 4) {
      const int64_t at = b * block_tokens, left = len - at;
      const uint64_t d = digest_of(tokens + t0 + at, left < block_tokens ? (int)left : block_tokens, lane);
      if (lane == 0) keys[k0 + b] = d;
    }
  }
}

// The rest of a queue of long prompts: blocks [0, first) of every request are digested; one workgroup a request chains them
// in its first wave while the others digest the blocks behind them, into LDS, in order.  A group of 16 digests is complete when
// its count says so; the chain waits for that, and only for waves of its own workgroup, which wait for nothing.
// Bound by the chain where `first` is large enough (see hash_with): a compute unit digests a block of 512 tokens in 0.15 us, a
// link takes 0.1.  Keys, launches of whole ranges / this, us: 64 prompts of 256 blocks of 512 tokens 30.5 / 28.3, 128 blocks
// 19.6 / 16.6; 200 prompts of 256 blocks 51.0 / 43.8; 128 of 59 20.8 / 18.4; 100 of 71 blocks of 128 tokens 21.1 / 18.9; 64 of
// 512 blocks of 256 tokens 53.2 / 54.0, the one of twelve batches that got slower.
constexpr int kPourBlocks = 4096;                         // most blocks of a request behind `first`
template <typename Tables>
__global__ __launch_bounds__(1024) void prefix_pour_kernel(const int32_t* __restrict__ tokens, const Tables off, int block_tokens,
                                                           int64_t first, uint64_t* keys) {
  __shared__ uint64_t digests[kPourBlocks];
  __shared__ int done[kPourBlocks / 16];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), waves = blockDim.x >> 6;
  const int r = blockIdx.x;
  const int64_t k0 = off.b[r], nk = off.b[r + 1] - k0;
  const int rest = nk > first ? (int)(nk - first) : 0;
  for (int g = threadIdx.x; g < kPourBlocks / 16; g += blockDim.x) done[g] = 0;
  __syncthreads();
  if (wave > 0) {
    const int64_t t0 = off.a[r], len = off.a[r + 1] - t0;
    for (int b = wave - 1; b < rest; b += waves - 1) {
      const int64_t at = (first + b) * block_tokens, left = len - at;
      const uint64_t d = digest_of(tokens + t0 + at, left < block_tokens ? (int)left : block_tokens, lane);
      if (lane == 0) {
        digests[b] = d;
        __hip_atomic_fetch_add(&done[b >> 4], 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
      }
    }
    return;
  }
  __builtin_amdgcn_s_setprio(3);                          // the chain is what the others are early for
  uint64_t salt = kFirstSalt;
  chain_range(keys + k0, keys + k0, 0, nk < first ? nk : first, salt, lane);
  // A group's digests are read once its count has been seen complete and a fence passed.  The count is read two groups ahead and
  // the digests one, before links that take longer than either; a group that was not complete by then is waited for.
  auto count = [&](int group) {
    return __hip_atomic_load(&done[group < kPourBlocks / 16 ? group : 0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  };
  auto digests_of = [&](int group) {
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    return digests[group * 16 + (lane & 15)];
  };
  int later = count(1);
  bool held = false;                                      // `ahead` are this group's
  uint64_t ahead = 0;
  for (int group = 0; group * 16 < rest; ++group) {
    const int left = rest - group * 16, n = left < 16 ? left : 16;
    if (!held) {
      while (__builtin_amdgcn_readfirstlane(count(group)) < n) __builtin_amdgcn_s_sleep(1);
      ahead = digests_of(group);
    }
    const uint64_t digest = ahead;
    held = left > 16 && __builtin_amdgcn_readfirstlane(later) >= (left < 32 ? left - 16 : 16);
    if (held) ahead = digests_of(group + 1);
    later = count(group + 2);
    uint32_t kl = 0, kh = 0;
    chain_four<0>(digest, salt, kl, kh);
    if (n > 4) chain_four<4>(digest, salt, kl, kh);
    if (n > 8) chain_four<8>(digest, salt, kl, kh);
    if (n > 12) chain_four<12>(digest, salt, kl, kh);
    if (lane < n) keys[k0 + first + group * 16 + lane] = ((uint64_t)kh << 32) | kl;
  }
}

// Does c[0 .. n), ascending, hold `key`?  Keys are hashes, spread evenly, so a probe tells not only on which side the key
// lies but about how far: the first guess is off by some sqrt(n) / 2 places (220 of 200000), the next by the root of that,
// and the rest is next to it: 4.6 probes instead of 18.  What has been read always brackets the key, so any ascending array
// gives the right answer; where kGuesses do not close in (keys that are far from evenly spread), the bracket is bisected.
// Distances turn into places at the rate between the last two probes, so keys that fill parts of the range evenly are found
// as fast (16 instances whose keys leave half the range empty, 64 requests: 16.2 us a call;
// 26.9 at the mean rate of the whole array, 23.1 by bisection).
// Distances go by the upper 32 bits of key differences: 64-bit conversions and windows of several keys a probe cost more
// vector instructions than they save in loads (256 keys of 64 requests in 16 instances of 209000:
// 16.6 us with them, 13.5 without; bisection 19.1).
constexpr int kGuesses = 8;
__device__ __forceinline__ bool holds(const uint64_t* __restrict__ c, int64_t n, uint64_t key) {
  if (n <= 0) return false;
  const uint64_t first = c[0], last = c[n - 1];
  if (key <= first || key >= last) return key == first || key == last;
  int64_t lo = 0, hi = n - 1;                            // c[lo] < key < c[hi]
  if (n <= (int64_t)1 << 30) {
    int l = 0, h = (int)n - 1;
    float per_key = (float)h / ((float)(uint32_t)((last - first) >> 32) + 1.f);
    auto upper = [](uint64_t x, uint64_t y) { return (float)(uint32_t)((x > y ? x - y : y - x) >> 32); };
    int at = (int)fminf(upper(key, first) * per_key + 0.5f, (float)h), was = 0;
    uint64_t v_was = first;
    for (int guess = 0; guess < kGuesses && h - l > 1; ++guess) {
      at = at <= l ? l + 1 : (at >= h ? h - 1 : at);
      const uint64_t v = c[at];
      if (v == key) return true;
      if (v < key) l = at; else h = at;
      // places per key between the last two probes, where they are far enough apart to tell
      const float span = upper(v, v_was), gone = (float)(at > was ? at - was : was - at);
      if (gone >= 16.f && span > 0.f) per_key = gone * __builtin_amdgcn_rcpf(span);
      was = at;
      v_was = v;
      const int off = (int)fminf(upper(key, v) * per_key + 0.5f, (float)h);
      at = v < key ? at + off : at - off;
    }
    lo = l;
    hi = h;
  }
  while (hi - lo > 1) {
    const int64_t mid = (lo + hi) >> 1;
    const uint64_t v = c[mid];
    if (v == key) return true;
    if (v < key) lo = mid; else hi = mid;
  }
  return false;
}

template <typename Tables>     // a: key offsets, b: cache offsets
__global__ __launch_bounds__(256) void prefix_match_kernel(const uint64_t* __restrict__ keys,
                                                           const uint64_t* __restrict__ cache_keys, const Tables off,
                                                           int n_inst, int32_t* __restrict__ prefix_len) {
  __shared__ int first_miss;
  const int inst = blockIdx.x, r = blockIdx.y;
  const int64_t k0 = off.a[r], nk = off.a[r + 1] - k0;
  const uint64_t* c = cache_keys + off.b[inst];
  const int64_t nc = off.b[inst + 1] - off.b[inst];
  if (threadIdx.x == 0) first_miss = (int)nk;
  __syncthreads();
  for (int64_t base = 0; base < nk; base += 256) {
    const int64_t i = base + threadIdx.x;
    // the first miss of a wave speaks for it (a lane each: 2.5 us more, they queue for one LDS word)
    const uint64_t missed = __builtin_amdgcn_ballot_w64(i < nk && !holds(c, nc, keys[k0 + i]));
    if (missed != 0 && (threadIdx.x & 63) == 0) atomicMin(&first_miss, (int)i + __builtin_ctzll(missed));
    __syncthreads();
    if (first_miss < base + 256) break;                  // uniform: everyone reads the same value after the barrier
    __syncthreads();
  }
  if (threadIdx.x == 0) prefix_len[(int64_t)r * n_inst + inst] = first_miss;
}

// Few keys and instances (at most kSmallMatch pairs in any request): one workgroup per request looks all of them up, one a
// thread, and takes the best instance itself.
constexpr int kSmallMatch = 1024;
template <typename Tables>     // a: key offsets, b: cache offsets
__global__ __launch_bounds__(kSmallMatch) void prefix_small_match_kernel(const uint64_t* __restrict__ keys,
                                                                         const uint64_t* __restrict__ cache_keys,
                                                                         const Tables off, int n_inst,
                                                                         int32_t* __restrict__ prefix_len,
                                                                         int32_t* __restrict__ best_len,
                                                                         int32_t* __restrict__ best_inst) {
  __shared__ int first_miss[64];
  const int r = blockIdx.x, t = threadIdx.x;
  const int64_t k0 = off.a[r];
  const int nk = (int)(off.a[r + 1] - k0);
  if (t < n_inst) first_miss[t] = nk;
  __syncthreads();
  if (t < nk * n_inst) {
    const int inst = t / nk, i = t - inst * nk;
    const int64_t c0 = off.b[inst];
    if (!holds(cache_keys + c0, off.b[inst + 1] - c0, keys[k0 + i])) atomicMin(&first_miss[inst], i);
  }
  __syncthreads();
  if (t >= 64) return;
  const int mine = t < n_inst ? first_miss[t] : -1;
  if (t < n_inst) prefix_len[(int64_t)r * n_inst + t] = mine;
  int most = mine;
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) {
    const int other = __shfl_xor(most, d, 64);
    most = other > most ? other : most;
  }
  const uint64_t at = __builtin_amdgcn_ballot_w64(mine == most);          // the lowest of them
  if (t == 0) {
    best_len[r] = most;
    best_inst[r] = __builtin_ctzll(at);
  }
}

// Sixteen lanes per request read its row of prefix lengths side by side (one thread a request read it one by one; 64
// requests, 16 instances: a pass of keys and match 49.9 us before, 49.0 now).
constexpr int kBestLanes = 16;
__global__ __launch_bounds__(256) void prefix_best_kernel(const int32_t* __restrict__ prefix_len, int batch, int n_inst,
                                                          int32_t* __restrict__ best_len,
                                                          int32_t* __restrict__ best_inst) {
  const int r = blockIdx.x * (256 / kBestLanes) + threadIdx.x / kBestLanes, part = threadIdx.x % kBestLanes;
  int32_t len = 0, inst = n_inst > 0 ? 0 : -1;           // the longest, and of equals the first
  if (r < batch)
    for (int i = part; i < n_inst; i += kBestLanes) {
      const int32_t l = prefix_len[(int64_t)r * n_inst + i];
      if (l > len) {
        len = l;
        inst = i;
      }
    }
#pragma unroll
  for (int d = kBestLanes / 2; d >= 1; d >>= 1) {
    const int32_t l = __shfl_xor(len, d, 64), i = __shfl_xor(inst, d, 64);
    if (l > len || (l == len && i < inst)) {
      len = l;
      inst = i;
    }
  }
  if (r < batch && part == 0) {
    best_len[r] = len;
    best_inst[r] = inst;
  }
}

}  // namespace

namespace {

// Costs the split of a queue of long prompts rests on: one link of a chain, and the digest of one block when the whole chip
// digests - of 512 tokens, and of fewer about as much (a workgroup's start and the sum across the wave).  A rough figure does:
// the line only moves work between launches.  64 prompts, split into ranges / not at all / best of eleven splits, us: 1024 blocks
// of 16 tokens 92.5 / 101.9 / 91.7, 512 of 64 49.7 / 53.0 / 49.4, 256 of 512 31.3 / 32.7 / 30.4, 128 of 1024 22.6 / 21.5 /
// 21.1, 64 of 2048 (not split) 16.0 / 15.9 / 15.9.
constexpr double kChainNs = 95.0, kDigestNs = 0.64;
// ... and a block's digest on the compute unit that chains its request, per token and for the block (256 tokens 133 ns, 512 186):
// of 64, 80 and 110 for the block 80 was behind launches of whole ranges once, by 1.5 % (64 prompts of 512 blocks of 256 tokens
// 55.9, 54.0, 51.8 us, 53.2 by ranges; 256 prompts of 118 blocks of 512 29.2, 29.4, 31.1, 35.3).
constexpr double kUnitTokenNs = 0.207, kUnitBlockNs = 80.0;
constexpr int kComputeUnits = 256;

template <typename Tables>
hipError_t hash_with(const int32_t* tokens, const Tables& off, int batch, int block_tokens, int64_t max_blocks,
                     int64_t total_blocks, bool in_one_launch, uint64_t* keys, hipStream_t stream) {
  const unsigned cols = batch < 65535 ? (unsigned)batch : 65535u;          // the kernels stride over the rest
  // Few blocks and tokens per request: one launch.  14 blocks of 512 tokens: 3.0 + 3.5 us and a launch between them, now
  // 5.0 us; keys and match of that prompt 18.2 -> 14.8 us a pass.
  if (in_one_launch && max_blocks <= kShortHashBlocks) {
    const unsigned waves = max_blocks < 16 ? (unsigned)max_blocks : 16u;
    prefix_short_kernel<Tables><<<cols, waves * 64, 0, stream>>>(tokens, off, batch, block_tokens, keys);
    return hipGetLastError();
  }
  // Long prompts.  Where the digests of the whole queue take longer than another launch costs (about 4 us), only the first of
  // them get one; the rest are made beside the chain of their request, by its own compute unit.
  const double digest_ns = kDigestNs * (double)total_blocks;
  if (digest_ns >= 4000.0 && batch <= kComputeUnits) {
    const double unit_ns = kUnitBlockNs + kUnitTokenNs * block_tokens;
    const double behind = unit_ns > kChainNs ? (double)max_blocks * kChainNs / unit_ns : (double)max_blocks;
    const int64_t first = (max_blocks - (int64_t)behind + 15) & ~(int64_t)15;
    if (first < max_blocks && max_blocks - first <= kPourBlocks) {
      if (first > 0) {
        const int64_t quads = (first + 3) / 4;
        prefix_stage_kernel<Tables><<<dim3(cols, (unsigned)(quads < 8192 ? quads : 8192)), 256, 0, stream>>>(
            tokens, off, batch, block_tokens, Blocks{0, first}, Blocks{0, 0}, 0, keys);
      }
      prefix_pour_kernel<Tables><<<cols, 1024, 0, stream>>>(tokens, off, block_tokens, first, keys);
      return hipGetLastError();
    }
  }
  // Digests, then chains.  In a queue of more requests than compute units, or of more blocks than the LDS has room for, the
  // chains of the first blocks run beside the digests of the rest in a launch of their own: `first` is where both take equally
  // long.
  // 64 prompts of 256 blocks: 12 + 30 us unsplit, by ranges 6 + 11 + 20 (59.9 -> 54.7 us a pass with the match; 54.8 with
  // first = 112 instead of 64).
  int64_t first = (int64_t)(digest_ns / (kChainNs + kDigestNs * batch)) & ~(int64_t)15;
  if (digest_ns < 4000.0 || first == 0 || first + 32 > max_blocks) first = max_blocks;
  auto stage = [&](Blocks digest, Blocks chain) {
    const int chains = chain.lo < chain.hi ? 1 : 0;
    const int64_t quads = (digest.hi - digest.lo + 3) / 4;
    const unsigned rows = (unsigned)(quads < 8192 ? quads : 8192);         // and over these
    prefix_stage_kernel<Tables><<<dim3(cols, rows + chains), rows > 0 ? 256 : 64, 0, stream>>>(
        tokens, off, batch, block_tokens, digest, chain, chains, keys);
  };
  stage({0, first}, {0, 0});
  if (first < max_blocks) stage({first, max_blocks}, {0, first});
  stage({0, 0}, {first < max_blocks ? first : 0, max_blocks});
  return hipGetLastError();
}

template <typename Tables>
hipError_t match_with(const uint64_t* keys, const Tables& off, int batch, int64_t max_keys, const uint64_t* cache_keys,
                      int n_inst, int32_t* prefix_len, int32_t* best_len, int32_t* best_inst, hipStream_t stream) {
  // one launch where a workgroup per request has a thread for every pair (14 keys, 4 instances: 4.7 us, a launch
  // and 2, now 4.0; keys and match of that prompt 15.5 -> 12.1 us a pass); otherwise a workgroup per pair of
  // request and instance, and the best of each request after them
  if (n_inst >= 1 && n_inst <= 64 && max_keys * n_inst <= kSmallMatch) {
    const unsigned most = (unsigned)(max_keys * n_inst), threads = most < 64 ? 64u : (most + 63) / 64 * 64;
    prefix_small_match_kernel<Tables><<<(unsigned)batch, threads, 0, stream>>>(keys, cache_keys, off, n_inst, prefix_len,
                                                                              best_len, best_inst);
    return hipGetLastError();
  }
  if (n_inst > 0)
    prefix_match_kernel<Tables><<<dim3((unsigned)n_inst, (unsigned)batch), 256, 0, stream>>>(keys, cache_keys, off, n_inst,
                                                                                            prefix_len);
  const unsigned per = 256 / kBestLanes;
  prefix_best_kernel<<<((unsigned)batch + per - 1) / per, 256, 0, stream>>>(prefix_len, batch, n_inst, best_len, best_inst);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_prefix_hash(const int32_t* tokens, const PrefixTables& tables, int batch, int block_tokens,
                              int64_t max_blocks, int64_t total_blocks, bool in_one_launch, uint64_t* keys,
                              hipStream_t stream) {
  (void)hipGetLastError();
  if (tables.arg != nullptr)
    return hash_with(tokens, *tables.arg, batch, block_tokens, max_blocks, total_blocks, in_one_launch, keys, stream);
  return hash_with(tokens, TablePtrs{tables.a, tables.b}, batch, block_tokens, max_blocks, total_blocks, in_one_launch, keys, stream);
}

hipError_t launch_prefix_match(const uint64_t* keys, const PrefixTables& tables, int batch, int64_t max_keys,
                               const uint64_t* cache_keys, int n_inst, int32_t* prefix_len, int32_t* best_len,
                               int32_t* best_inst, hipStream_t stream) {
  (void)hipGetLastError();
  if (tables.arg != nullptr)
    return match_with(keys, *tables.arg, batch, max_keys, cache_keys, n_inst, prefix_len, best_len, best_inst, stream);
  return match_with(keys, TablePtrs{tables.a, tables.b}, batch, max_keys, cache_keys, n_inst, prefix_len, best_len, best_inst,
                    stream);
}

}  // namespace mc
