// Typed eviction order of one memory tier (Sec. 4.3.2, typed offloading).
//
// Each KV block carries its program's type label (busy = GPU queue, idle =
// CPU queue, inactive = Waiting) and its last access time.  A tier evicts by
// type first, in tier-reversed order (GPU: inactive, idle, busy; CPU:
// inactive, busy, idle), least recently used first within a type, equal
// (type, time) lowest block id first.  That is one ascending sort of the
// 64-bit key (type position << 62 | last access), equal keys by block id,
// followed by the bytes freed along that order and the number of evictions
// that frees the requested bytes.  The pair (key, id) is unique, so any way of
// sorting gives the same order.  Three forms by block count, each bound by the
// latency of its chain of launches rather than by bandwidth (a call reads and
// writes 25 B a block):
//
//   direct  (up to DIRECT_MAX) one kernel: every workgroup stages all keys in
//           LDS and each wave counts, for its blocks, the blocks before it and
//           their bytes, which are the block's place and its prefix; no
//           workgroup waits for another.
//   buckets (up to BUCKET_MAX) four or five kernels: a sorted pseudo-random
//           sample gives up to 1024 buckets of similar size, whatever the
//           layout of keys and ties (evict_split.h); the blocks of each bucket
//           are counted, gathered and sorted in LDS by one workgroup, which
//           knows from the bucket totals where its bucket begins.
//   radix   (above) a device-wide stable LSD radix sort:
//     keys     build keys, validate, OR/AND of all keys;
//     per pass (8-bit digit, 8 passes; a digit on which every key agrees needs
//     no pass, and each kernel works out from the OR/AND which of the two
//     key/value buffers holds the current order, so such a pass is empty
//     launches and no memory traffic), one workgroup per tile:
//     - hist: per tile, a 256-bin histogram -> hist[digit][tile];
//     - dscan: one workgroup per digit, an exclusive scan of that digit's
//       counts over the tiles and the digit's total;
//     - scatter: the stable rank of every key among the tile's keys of its
//       digit (wave64 ballots over the 8 digit bits rank it within its wave's
//       64 keys of a slice, one scan per digit over (slice, wave) in LDS orders
//       the groups as the keys were ordered); position = digit base + keys of
//       the digit in lower tiles + that rank;
//     prefix   inclusive u64 scan of block bytes in eviction order (tile scans,
//              then a fix-up whose workgroups each sum the tile totals below
//              their tile, or above FIX_SCAN_TILES a one-workgroup scan of the
//              tile totals first) and the eviction count.
//
// The workspace is the caller's, so nothing is allocated here.
#include "evict_split.h"
#include "mori_internal.h"
#include "sort.h"
#include "wave.h"

namespace mori {
namespace {

constexpr int ET = EVICT_WG;            // threads per tile workgroup
constexpr int ENW = ET / 64;            // waves per tile workgroup
constexpr int EIPT = EVICT_KEYS_PER_THREAD;  // keys per thread of a radix tile (measured against 4)
constexpr uint64_t TIME_LIMIT = 1ull << 62;
constexpr uint32_t KEY_WG_MAX = 128;    // workgroups of the keys kernel at most (more: same-address atomics)
constexpr int KEYS_PER_ROUND = 8;       // keys per thread whose loads the keys kernel issues together
// Tile counts up to this finish the prefix with one kernel (every workgroup
// reads the tile totals: 8 B each) instead of a tile scan, a fix-up and a
// result kernel.
constexpr uint32_t FIX_SCAN_TILES = 1024;

// Direct and bucket forms: workgroups of 1024 threads.  Measured per call
// (sizes given, half the blocks tied), the form before -> this one:
//   blocks     4 096   8 192   16 384   69 938   262 144   2^20
//   us         60->8   66->15  70->22   86->27   114->36   178->67
constexpr int BT = 1024, BNW = BT / 64;
constexpr uint32_t DIRECT_WG = 256;         // one per compute unit
constexpr int SAMPLE_WG = 64;
constexpr int BUCKET_IPT = BUCKET_CAP / BT;  // entries per thread that sorts a bucket
static_assert(BUCKET_CAP % BT == 0, "whole entries per thread");
// Blocks per thread of the partition kernels: one while that leaves a workgroup
// for each compute unit, two above (2^20 blocks: 2 us faster than one or four).
constexpr uint32_t PARTITION_ONE_MAX = 1u << 18;

struct EvictArgs {
  uint32_t N, ntiles, tier;
  const uint8_t* type;
  const uint64_t* last_access;
  const uint32_t* size;
  uint64_t unit_bytes, need;
  uint64_t* keys[2];
  uint32_t* vals[2];
  uint32_t* hist;       // [256][ntiles]
  uint32_t* dtot;       // [256] keys per digit
  uint64_t* tile_sum;   // [ntiles]
  uint64_t* misc;       // [0] OR of keys, [1] AND of keys, [2] error bits, [3] evictions short of need
  uint32_t* order;      // out [N]
  uint64_t* prefix;     // out [N] (or workspace)
  uint32_t* result;     // out [2]: count, error bits
};

// A block's key; invalid metadata (reported separately) gives some key.
__device__ inline uint64_t block_key(uint32_t tier, uint32_t type, uint64_t last_access) {
  // position of each type label in the tier's eviction order: GPU inactive,
  // idle, busy; CPU inactive, busy, idle
  const uint32_t pos = tier == MORI_TIER_GPU ? 2u - min(type, 2u) : type == MORI_TYPE_BUSY ? 1u
                       : type == MORI_TYPE_IDLE ? 2u : 0u;
  return ((uint64_t)pos << 62) | (last_access & (TIME_LIMIT - 1));
}
__device__ inline uint64_t block_error(uint32_t type, uint64_t last_access) {
  return type > MORI_TYPE_INACTIVE || last_access >= TIME_LIMIT ? MORI_DEV_BAD_BLOCK : 0u;
}

__global__ void evict_init_kernel(EvictArgs a) {
  a.misc[0] = 0;
  a.misc[1] = ~0ull;
  a.misc[2] = 0;
  a.misc[3] = 0;
}

__global__ __launch_bounds__(ET) void evict_keys_kernel(EvictArgs a) {
  uint64_t o = 0, n = ~0ull, err = 0;
  // rounds of KEYS_PER_ROUND keys per thread, all their loads issued first
  for (uint64_t i0 = (uint64_t)blockIdx.x * ET * KEYS_PER_ROUND; i0 < a.N;
       i0 += (uint64_t)gridDim.x * ET * KEYS_PER_ROUND) {
    uint8_t typ[KEYS_PER_ROUND];
    uint64_t la[KEYS_PER_ROUND];
#pragma unroll
    for (int u = 0; u < KEYS_PER_ROUND; ++u) {
      const uint64_t i = i0 + (uint64_t)u * ET + threadIdx.x;
      typ[u] = i < a.N ? a.type[i] : 0;
      la[u] = i < a.N ? a.last_access[i] : 0;
    }
#pragma unroll
    for (int u = 0; u < KEYS_PER_ROUND; ++u) {
      const uint64_t i = i0 + (uint64_t)u * ET + threadIdx.x;
      if (i >= a.N) continue;
      err |= block_error(typ[u], la[u]);
      const uint64_t key = block_key(a.tier, typ[u], la[u]);
      a.keys[0][i] = key;
      a.vals[0][i] = (uint32_t)i;
      o |= key;
      n &= key;
    }
  }
  // wave, then workgroup reduction: one set of global atomics per workgroup
  __shared__ uint64_t s_red[3][ENW];
  o = wave::all_or<uint64_t>(o);
  n = wave::all_and<uint64_t>(n);
  err = wave::all_or<uint64_t>(err);
  const int wid = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
    s_red[0][wid] = o;
    s_red[1][wid] = n;
    s_red[2][wid] = err;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < ENW; ++w) {
      o |= s_red[0][w];
      n &= s_red[1][w];
      err |= s_red[2][w];
    }
    atomicOr((unsigned long long*)&a.misc[0], (unsigned long long)o);
    atomicAnd((unsigned long long*)&a.misc[1], (unsigned long long)n);
    if (err) atomicOr((unsigned long long*)&a.misc[2], (unsigned long long)err);
  }
}

__device__ inline uint64_t varying_bits(const EvictArgs& a) { return a.misc[0] ^ a.misc[1]; }

__device__ inline bool digit_varies(const EvictArgs& a, int shift) {
  return ((varying_bits(a) >> shift) & 255u) != 0;
}

// Which buffer holds the order before the pass at `shift`: passes over
// constant digits are skipped, so it is the parity of the varying digits below.
__device__ inline int source_buffer(const EvictArgs& a, int shift) {
  const uint64_t v = varying_bits(a);
  int n = 0;
  for (int s = 0; s < shift; s += 8) n += ((v >> s) & 255u) != 0;
  return n & 1;
}

__global__ __launch_bounds__(ET) void evict_hist_kernel(EvictArgs a, int shift) {
  __shared__ uint32_t s_h[256];
  if (a.misc[2] || !digit_varies(a, shift)) return;
  s_h[threadIdx.x] = 0;
  __syncthreads();
  const uint64_t* k = a.keys[source_buffer(a, shift)];
  const uint64_t base = (uint64_t)blockIdx.x * (ET * EIPT);
  const uint64_t lanemask_lt = (1ull << (threadIdx.x & 63)) - 1ull;
#pragma unroll
  for (int it = 0; it < EIPT; ++it) {
    // keys of a program share their time, so digits repeat within a wave: one
    // LDS increment per distinct digit (its first lane adds the group's size)
    const uint64_t i = base + it * ET + threadIdx.x;
    const bool valid = i < a.N;
    const uint32_t d = valid ? (uint32_t)(k[i] >> shift) & 255u : 0u;
    const uint64_t same = __ballot(valid) & ~wave::digit_differs<8>(d);
    if (valid && (same & lanemask_lt) == 0) atomicAdd(&s_h[d], (uint32_t)__popcll(same));
  }
  __syncthreads();
  a.hist[(uint64_t)threadIdx.x * a.ntiles + blockIdx.x] = s_h[threadIdx.x];
}

// Block-wide exclusive scan of one u32 per thread (256 threads); *total gets the sum.
__device__ inline uint32_t scan256(uint32_t v, uint32_t* s_w, uint32_t* total) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const uint32_t x = wave::incl_add(v);
  if (lane == 63) s_w[wid] = x;
  __syncthreads();
  uint32_t before = 0, all = 0;
#pragma unroll
  for (int w = 0; w < ENW; ++w) {
    before += w < wid ? s_w[w] : 0u;
    all += s_w[w];
  }
  __syncthreads();
  *total = all;
  return before + x - v;
}

// The tile's keys to their global positions, staged through LDS in the
// tile's digit order so that each wave's stores cover a few contiguous runs
// (one per digit it meets) instead of one scattered 8-byte store per lane.
// s_tstart[d]: first tile-local slot of digit d; s_off[d]: its global slot;
// s_cnt: the (slice, wave, digit) offsets within each digit; n: valid keys.
// Every thread calls it; it begins and ends with a barrier.
__device__ void store_tile(const uint64_t (&key)[EIPT], const uint32_t (&val)[EIPT], const uint32_t (&dig)[EIPT],
                           const uint32_t (&rnk)[EIPT], const uint16_t (*s_cnt)[ENW][256], const uint32_t* s_tstart,
                           const uint32_t* s_off, uint64_t* s_k, uint32_t* s_v, uint32_t n, int shift, uint64_t* kd,
                           uint32_t* vd) {
  const int tid = threadIdx.x, wid = tid >> 6;
  __syncthreads();
#pragma unroll
  for (int it = 0; it < EIPT; ++it) {
    const uint32_t d = dig[it];
    if (d < 256u) {
      const uint32_t local = s_tstart[d] + s_cnt[it][wid][d] + rnk[it];
      s_k[local] = key[it];
      s_v[local] = val[it];
    }
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < EIPT; ++j) {
    const uint32_t local = j * ET + tid;
    if (local < n) {
      const uint64_t k = s_k[local];
      const uint32_t d = (uint32_t)(k >> shift) & 255u;
      const uint32_t pos = s_off[d] + (local - s_tstart[d]);
      kd[pos] = k;
      vd[pos] = s_v[local];
    }
  }
}

// One workgroup per digit: exclusive scan of hist[digit][0..ntiles) in place
// and the digit's total.
__global__ __launch_bounds__(ET) void evict_dscan_kernel(EvictArgs a, int shift) {
  __shared__ uint32_t s_w[ENW];
  if (a.misc[2] || !digit_varies(a, shift)) return;
  uint32_t* h = a.hist + (uint64_t)blockIdx.x * a.ntiles;
  uint32_t carry = 0;
  for (uint32_t t0 = 0; t0 < a.ntiles; t0 += ET) {
    const uint32_t t = t0 + threadIdx.x;
    const uint32_t v = t < a.ntiles ? h[t] : 0u;
    uint32_t tot;
    const uint32_t ex = scan256(v, s_w, &tot);
    if (t < a.ntiles) h[t] = carry + ex;
    carry += tot;
  }
  if (threadIdx.x == 0) a.dtot[blockIdx.x] = carry;
}

__global__ __launch_bounds__(ET) void evict_scatter_kernel(EvictArgs a, int shift) {
  // s_cnt[slice][wave][digit]: keys of that digit in that wave's 64 keys of the
  // slice, then (after the per-digit scan) their offset within the tile
  __shared__ uint16_t s_cnt[EIPT][ENW][256];
  __shared__ uint32_t s_off[256];     // this tile's global base per digit
  __shared__ uint32_t s_tstart[256];  // ... and its first slot within the tile
  __shared__ uint64_t s_k[ET * EIPT];
  __shared__ uint32_t s_v[ET * EIPT];
  __shared__ uint32_t s_w[ENW];
  if (a.misc[2] || !digit_varies(a, shift)) return;
  const int src = source_buffer(a, shift);
  const uint64_t* ks = a.keys[src];
  const uint32_t* vs = a.vals[src];
  uint64_t* kd = a.keys[src ^ 1];
  uint32_t* vd = a.vals[src ^ 1];
  const uint64_t base = (uint64_t)blockIdx.x * (ET * EIPT);
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  uint32_t tot;
  const uint32_t before = a.hist[(uint64_t)tid * a.ntiles + blockIdx.x];  // scanned by evict_dscan_kernel
  const uint32_t total_d = a.dtot[tid];
  const uint32_t digit_base = scan256(total_d, s_w, &tot);
  s_off[tid] = digit_base + before;
#pragma unroll
  for (int it = 0; it < EIPT; ++it)
#pragma unroll
    for (int w = 0; w < ENW; ++w) s_cnt[it][w][tid] = 0;
  __syncthreads();
  // rank of every key among the keys of its digit in its wave's slice (ballots)
  const uint64_t lanemask_lt = (1ull << lane) - 1ull;
  uint64_t key[EIPT];
  uint32_t val[EIPT], dig[EIPT], rnk[EIPT];
#pragma unroll
  for (int it = 0; it < EIPT; ++it) {
    const uint64_t i = base + it * ET + tid;
    const bool valid = i < a.N;
    key[it] = valid ? ks[i] : 0ull;
    val[it] = valid ? vs[i] : 0u;
    const uint32_t d = (uint32_t)(key[it] >> shift) & 255u;
    const uint64_t same = __ballot(valid) & ~wave::digit_differs<8>(d);
    const uint32_t r = __popcll(same & lanemask_lt);
    if (valid && r == 0) s_cnt[it][wid][d] = (uint16_t)__popcll(same);
    dig[it] = valid ? d : 256u;
    rnk[it] = r;
  }
  __syncthreads();
  uint32_t run = 0;  // per digit (one per thread): offsets in (slice, wave) order, i.e. original key order
#pragma unroll
  for (int it = 0; it < EIPT; ++it)
#pragma unroll
    for (int w = 0; w < ENW; ++w) {
      const uint32_t c = s_cnt[it][w][tid];
      s_cnt[it][w][tid] = (uint16_t)run;
      run += c;
    }
  uint32_t n;
  s_tstart[tid] = scan256(run, s_w, &n);
  store_tile(key, val, dig, rnk, s_cnt, s_tstart, s_off, s_k, s_v, n, shift, kd, vd);
}

// Inclusive scan of freed bytes within each tile; tile totals to tile_sum.
// Global memory is read and written in striped (coalesced) order and the
// blocked per-thread scan runs on an LDS copy of the tile.
__global__ __launch_bounds__(ET) void evict_prefix_tiles_kernel(EvictArgs a) {
  __shared__ uint64_t s_b[ET * EIPT];
  __shared__ uint64_t s_w[ENW + 1];
  if (a.misc[2]) return;
  const uint32_t* order = a.vals[source_buffer(a, 64)];
  const uint64_t base = (uint64_t)blockIdx.x * (ET * EIPT);
  const int tid = threadIdx.x;
#pragma unroll
  for (int it = 0; it < EIPT; ++it) {
    const uint64_t i = base + it * ET + tid;
    uint64_t bytes = 0;
    if (i < a.N) {
      const uint32_t b = order[i];
      a.order[i] = b;
      bytes = (uint64_t)(a.size ? a.size[b] : 1u) * a.unit_bytes;
    }
    s_b[it * ET + tid] = bytes;
  }
  __syncthreads();
  uint64_t v[EIPT];
  uint64_t sum = 0;
#pragma unroll
  for (int j = 0; j < EIPT; ++j) {  // blocked: keys tid * EIPT .. + EIPT - 1 of the tile
    sum += s_b[tid * EIPT + j];
    v[j] = sum;
  }
  // exclusive scan of the per-thread totals
  const int lane = tid & 63, wid = tid >> 6;
  const uint64_t x = wave::incl_add(sum);
  if (lane == 63) s_w[wid] = x;
  __syncthreads();
  if (tid == 0) {
    uint64_t run = 0;
    for (int w = 0; w < ENW; ++w) {
      const uint64_t c = s_w[w];
      s_w[w] = run;
      run += c;
    }
    s_w[ENW] = run;
  }
  __syncthreads();
  const uint64_t before = s_w[wid] + x - sum;
#pragma unroll
  for (int j = 0; j < EIPT; ++j) s_b[tid * EIPT + j] = before + v[j];
  __syncthreads();
#pragma unroll
  for (int it = 0; it < EIPT; ++it) {
    const uint64_t i = base + it * ET + tid;
    if (i < a.N) a.prefix[i] = s_b[it * ET + tid];
  }
  if (tid == 0) a.tile_sum[blockIdx.x] = s_w[ENW];
}

__global__ __launch_bounds__(1024) void evict_prefix_top_kernel(EvictArgs a) {
  __shared__ uint64_t s_w[1024 / 64 + 1];
  if (a.misc[2]) return;
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  uint64_t carry = 0;
  for (uint32_t t0 = 0; t0 < a.ntiles; t0 += 1024) {
    const uint32_t t = t0 + threadIdx.x;
    const uint64_t v = t < a.ntiles ? a.tile_sum[t] : 0ull;
    const uint64_t x = wave::incl_add(v);
    if (lane == 63) s_w[wid] = x;
    __syncthreads();
    if (wid == 0) {
      const uint64_t w = lane < 16 ? s_w[lane] : 0ull;
      const uint64_t wi = wave::incl_add(w);
      if (lane < 16) s_w[lane] = wi - w;
      if (lane == 15) s_w[16] = wi;
    }
    __syncthreads();
    if (t < a.ntiles) a.tile_sum[t] = carry + s_w[wid] + x - v;  // exclusive base of tile t
    carry += s_w[16];
    __syncthreads();
  }
}

__global__ __launch_bounds__(ET) void evict_prefix_fix_kernel(EvictArgs a) {
  if (a.misc[2]) return;
  const uint64_t add = a.tile_sum[blockIdx.x];
  const uint64_t base = (uint64_t)blockIdx.x * (ET * EIPT);
  uint32_t short_of_need = 0;
  for (int it = 0; it < EIPT; ++it) {
    const uint64_t i = base + it * ET + threadIdx.x;
    if (i < a.N) {
      const uint64_t p = a.prefix[i] + add;
      a.prefix[i] = p;
      short_of_need += p < a.need;
    }
  }
  __shared__ uint32_t s_short[ENW];
  short_of_need = wave::sum(short_of_need);
  if ((threadIdx.x & 63) == 0) s_short[threadIdx.x >> 6] = short_of_need;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t t = 0;
    for (int w = 0; w < ENW; ++w) t += s_short[w];
    if (t) atomicAdd((unsigned long long*)&a.misc[3], (unsigned long long)t);
  }
}

// Up to FIX_SCAN_TILES tiles: the fix-up workgroups scan the tile totals
// themselves (each sums the totals below its tile) and the result comes from
// the one workgroup whose tile holds the first prefix >= need (the prefix never
// decreases, so that tile is unique; without one, the last tile's workgroup
// reports every block), so neither the one-workgroup tile scan nor the result
// kernel runs.
__global__ __launch_bounds__(ET) void evict_prefix_fix_scan_kernel(EvictArgs a) {
  __shared__ uint64_t s_red[ENW][2];
  if (a.misc[2]) {
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      a.result[0] = 0;
      a.result[1] = (uint32_t)a.misc[2];
    }
    return;
  }
  uint64_t below = 0, all = 0;  // totals of the tiles below this one, and of every tile
  for (uint32_t t = threadIdx.x; t < a.ntiles; t += ET) {
    const uint64_t v = a.tile_sum[t];
    if (t < blockIdx.x) below += v;
    all += v;
  }
  below = wave::sum(below);
  all = wave::sum(all);
  if ((threadIdx.x & 63) == 0) {
    s_red[threadIdx.x >> 6][0] = below;
    s_red[threadIdx.x >> 6][1] = all;
  }
  __syncthreads();
  below = all = 0;
#pragma unroll
  for (int w = 0; w < ENW; ++w) {
    below += s_red[w][0];
    all += s_red[w][1];
  }
  const uint64_t base = (uint64_t)blockIdx.x * (ET * EIPT);
  uint32_t short_of_need = 0;
  for (int it = 0; it < EIPT; ++it) {
    const uint64_t i = base + it * ET + threadIdx.x;
    if (i < a.N) {
      const uint64_t p = a.prefix[i] + below;
      a.prefix[i] = p;
      short_of_need += p < a.need;
    }
  }
  __syncthreads();  // s_red is reused
  short_of_need = wave::sum(short_of_need);
  if ((threadIdx.x & 63) == 0) s_red[threadIdx.x >> 6][0] = short_of_need;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint64_t c = 0;
    for (int w = 0; w < ENW; ++w) c += s_red[w][0];
    const uint64_t len = a.N - base < (uint64_t)(ET * EIPT) ? a.N - base : (uint64_t)(ET * EIPT);
    const bool last = blockIdx.x == a.ntiles - 1;
    if (blockIdx.x == 0) a.result[1] = 0;
    if (a.need == 0) {
      if (blockIdx.x == 0) a.result[0] = 0;
    } else if (below < a.need && c < len) {  // the first prefix >= need is in this tile
      a.result[0] = (uint32_t)(base + c + 1);
    } else if (last && all < a.need) {  // no prefix reaches need: every block
      a.result[0] = a.N;
    }
  }
}

__global__ void evict_result_kernel(EvictArgs a) {
  const uint64_t err = a.misc[2];
  uint64_t count = 0;
  if (!err && a.need > 0) {
    count = a.misc[3] + 1;  // freed bytes are non-decreasing along the order
    if (count > a.N) count = a.N;
  }
  a.result[0] = (uint32_t)count;
  a.result[1] = (uint32_t)err;
}

// ---- direct and bucket forms ------------------------------------------------

// One block's entry of the order, its prefix (`through` = bytes freed up to and
// with it) and, where the prefix first reaches need, the eviction count.
__device__ inline void emit(const EvictArgs& a, uint32_t rank, uint32_t id, uint64_t through, uint64_t own) {
  a.order[rank] = id;
  if (a.prefix) a.prefix[rank] = through;
  if (through >= a.need && through - own < a.need) a.result[0] = rank + 1;
}

// The result's words that no block's entry decides.  One thread.
__device__ inline void finish_result(const EvictArgs& a, uint64_t err, uint64_t total) {
  a.result[1] = (uint32_t)err;
  if (err || a.need == 0) a.result[0] = 0;
  else if (total < a.need) a.result[0] = a.N;
}

// Up to DIRECT_MAX blocks, one launch.  Counting is quadratic but spread over
// every compute unit.
template <bool SIZES, int E>
__global__ __launch_bounds__(BT) void evict_direct_kernel(EvictArgs a) {
  __shared__ uint64_t s_key[DIRECT_MAX];
  __shared__ uint32_t s_size[SIZES ? DIRECT_MAX : 1];
  __shared__ uint32_t s_err;
  __shared__ uint64_t s_tot[BNW];
  const uint32_t tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const uint32_t chunks = (a.N + 64 * GROUP - 1) / (64 * GROUP) * GROUP;
  if (tid == 0) s_err = 0;
  __syncthreads();
  uint64_t err = 0, units = 0;
  constexpr int U = 4;  // blocks per thread whose loads are in flight together
  for (uint32_t j0 = tid; j0 < chunks * 64; j0 += U * BT) {
    uint32_t ty[U], sz[U];
    uint64_t la[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t j = min(j0 + u * BT, a.N - 1);
      ty[u] = a.type[j];
      la[u] = a.last_access[j];
      sz[u] = SIZES ? a.size[j] : 1u;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t j = j0 + u * BT;
      if (j >= chunks * 64) break;
      const bool valid = j < a.N;
      if (valid) {
        err |= block_error(ty[u], la[u]);
        units += sz[u];
      }
      s_key[j] = valid ? block_key(a.tier, ty[u], la[u]) : ~0ull;
      if (SIZES) s_size[j] = valid ? sz[u] : 0u;
    }
  }
  if (err) atomicOr(&s_err, (uint32_t)err);
  units = wave::sum(units);
  if (lane == 0) s_tot[wid] = units;
  __syncthreads();
  if (blockIdx.x == 0 && tid == 0) {
    uint64_t total = 0;
    for (int w = 0; w < BNW; ++w) total += s_tot[w];
    finish_result(a, s_err, total * a.unit_bytes);
  }
  if (s_err) return;
  const uint32_t waves = gridDim.x * BNW;
  for (uint32_t i0 = (blockIdx.x * BNW + wid) * E; i0 < a.N; i0 += E * waves) {
    uint32_t rank[E];
    uint64_t before[E];
    count_before<E, SIZES>(s_key, s_size, chunks, i0, rank, before);
#pragma unroll
    for (int e = 0; e < E; ++e)
      if (lane == 0 && i0 + e < a.N) {
        const uint64_t own = SIZES ? s_size[i0 + e] : 1u;
        emit(a, rank[e], i0 + e, (before[e] + own) * a.unit_bytes, own * a.unit_bytes);
      }
  }
}

__global__ void evict_empty_kernel(EvictArgs a) {
  a.result[0] = 0;
  a.result[1] = 0;
}

void launch_direct(const EvictArgs& a, hipStream_t s) {
  if (a.N == 0) {
    hipLaunchKernelGGL(evict_empty_kernel, dim3(1), dim3(1), 0, s, a);
    return;
  }
  const uint32_t wg = (a.N + BNW - 1) / BNW;
  const dim3 grid(wg < DIRECT_WG ? wg : DIRECT_WG);
  const bool one = a.N <= DIRECT_WG * BNW;  // one block a wave, else two that share their LDS reads
  if (a.size && one) hipLaunchKernelGGL((evict_direct_kernel<true, 1>), grid, dim3(BT), 0, s, a);
  else if (a.size) hipLaunchKernelGGL((evict_direct_kernel<true, 2>), grid, dim3(BT), 0, s, a);
  else if (one) hipLaunchKernelGGL((evict_direct_kernel<false, 1>), grid, dim3(BT), 0, s, a);
  else hipLaunchKernelGGL((evict_direct_kernel<false, 2>), grid, dim3(BT), 0, s, a);
}

struct BucketArgs {
  EvictArgs e;
  uint32_t B, S;       // buckets (a power of two), samples (a multiple of B)
  uint64_t* spl_key;   // [B - 1] splitters, ascending (key, id): bucket b holds the blocks from
  uint32_t* spl_id;    //         splitter b - 1 up to, without, splitter b
  uint64_t* sample;    // [S] sampled keys
  uint32_t* count;     // [B] blocks per bucket
  uint32_t* taken;     // [B] places handed out so far
  uint64_t* units;     // [B] size units per bucket (with sizes)
  uint32_t* first;     // [B + 1] blocks below each bucket
  uint64_t* below;     // [B + 1] size units below each bucket
  uint32_t* over;      // 1: some bucket is larger than BUCKET_CAP
  uint64_t* err;       // device error bits
  uint64_t* key;       // [N] keys, bucket by bucket
  uint32_t* id;        // [N] block ids, bucket by bucket
};

__device__ inline void clear_buckets(const BucketArgs& a) {
  for (uint32_t b = threadIdx.x; b < a.B; b += BT) {
    a.count[b] = 0;
    a.taken[b] = 0;
    a.units[b] = 0;
  }
  if (threadIdx.x == 0) {
    *a.err = 0;
    *a.over = 0;
  }
}

// The sampled keys, gathered once: the splitter kernel's workgroups then read
// them as one stretch instead of each gathering all of them line by line.
__global__ __launch_bounds__(SAMPLE_WG) void evict_sample_kernel(BucketArgs a) {
  const uint32_t j = blockIdx.x * SAMPLE_WG + threadIdx.x;
  if (j >= a.S) return;
  const uint32_t i = sample_block(j, a.S, a.e.N);
  a.sample[j] = block_key(a.e.tier, a.e.type[i], a.e.last_access[i]);
}

// Splitters: every workgroup stages the whole sample and ranks its share;
// every S / B-th sample is a splitter.  Also clears what the next kernels add to.
template <int E, bool GATHERED>
__global__ __launch_bounds__(BT) void evict_splitter_kernel(BucketArgs a) {
  __shared__ uint64_t s_key[SAMPLES_MAX];
  const uint32_t tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  if (blockIdx.x == 0) clear_buckets(a);
  if constexpr (GATHERED) {
    for (uint32_t j = tid; j < a.S; j += BT) s_key[j] = a.sample[j];
  } else {
    constexpr int U = 4;
    for (uint32_t j0 = tid; j0 < a.S; j0 += U * BT) {
      uint32_t ty[U];
      uint64_t la[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const uint32_t i = sample_block(min(j0 + u * BT, a.S - 1), a.S, a.e.N);
        ty[u] = a.e.type[i];
        la[u] = a.e.last_access[i];
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (j0 + u * BT < a.S) s_key[j0 + u * BT] = block_key(a.e.tier, ty[u], la[u]);
    }
  }
  __syncthreads();
  const uint32_t waves = gridDim.x * BNW, every = a.S / a.B;
  for (uint32_t j0 = (blockIdx.x * BNW + wid) * E; j0 < a.S; j0 += E * waves) {
    uint32_t rank[E];
    uint64_t unused[E];
    count_before<E, false>(s_key, nullptr, a.S / 64, j0, rank, unused);
#pragma unroll
    for (int e = 0; e < E; ++e)
      if (lane == 0 && rank[e] && rank[e] % every == 0) {
        a.spl_key[rank[e] / every - 1] = s_key[j0 + e];
        a.spl_id[rank[e] / every - 1] = sample_block(j0 + e, a.S, a.e.N);
      }
  }
}

// Bucket of (key, id): the number of splitters at or below it.
__device__ inline uint32_t find_bucket(const uint64_t* s_key, const uint32_t* s_id, uint32_t B, uint64_t key,
                                       uint32_t id) {
  uint32_t pos = 0;
  for (uint32_t step = B >> 1; step; step >>= 1) {
    const uint64_t k = s_key[pos + step - 1];
    if (k < key || (k == key && s_id[pos + step - 1] <= id)) pos += step;
  }
  return pos;
}

// Exclusive scan over the workgroup's 1024 threads; *total gets the sum.
template <typename T>
__device__ inline T scan_wg(T v, T* s_w, T* total) {
  const uint32_t lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const T x = wave::incl_add(v);
  if (lane == 63) s_w[wid] = x;
  __syncthreads();
  const T w = lane < BNW ? s_w[lane] : T(0);
  const T below = wave::sum(lane < wid ? w : T(0));
  *total = wave::sum(w);
  __syncthreads();
  return below + x - v;
}

// Partition, IPT blocks per thread.  COUNT: blocks and size units per bucket,
// and the validation.  Otherwise every block's key and id to its bucket's
// stretch: workgroups reserve places in it in any order (the bucket is sorted
// afterwards).
template <int IPT, bool COUNT>
__global__ __launch_bounds__(BT) void evict_partition_kernel(BucketArgs a) {
  __shared__ uint64_t s_key[BUCKETS_MAX];
  __shared__ uint32_t s_id[BUCKETS_MAX];
  __shared__ uint32_t s_cnt[BUCKETS_MAX];
  __shared__ unsigned long long s_units[COUNT ? BUCKETS_MAX : 1];
  __shared__ uint32_t s_base[COUNT ? 1 : BUCKETS_MAX];
  __shared__ uint32_t s_w[BNW];
  const uint32_t tid = threadIdx.x;
  const uint64_t i0 = (uint64_t)blockIdx.x * (BT * IPT) + tid;
  uint32_t ty[IPT], sz[IPT];
  uint64_t la[IPT];
#pragma unroll
  for (int it = 0; it < IPT; ++it) {
    const uint32_t i = (uint32_t)min(i0 + it * BT, (uint64_t)a.e.N - 1);
    ty[it] = a.e.type[i];
    la[it] = a.e.last_access[i];
    sz[it] = COUNT && a.e.size ? a.e.size[i] : 0u;
  }
  if (tid < a.B) {
    s_key[tid] = tid + 1 < a.B ? a.spl_key[tid] : ~0ull;
    s_id[tid] = tid + 1 < a.B ? a.spl_id[tid] : 0u;
    s_cnt[tid] = 0;
    if (COUNT) s_units[tid] = 0;
  }
  __syncthreads();
  const uint32_t lane = tid & 63;
  const uint64_t lanemask_lt = (1ull << lane) - 1ull;
  uint32_t bkt[IPT], r[IPT], err = 0;
#pragma unroll
  for (int it = 0; it < IPT; ++it) {
    const uint64_t i = i0 + it * BT;
    const bool valid = i < a.e.N;
    if (COUNT && valid) err |= (uint32_t)block_error(ty[it], la[it]);
    la[it] = block_key(a.e.tier, ty[it], la[it]);
    bkt[it] = find_bucket(s_key, s_id, a.B, la[it], (uint32_t)i);
    r[it] = 0;
    // A program's blocks have neighbouring ids and times, so a wave's blocks
    // mostly share one or two buckets: those take one increment each, the
    // rest one a lane.
    uint64_t todo = __ballot(valid);
#pragma unroll
    for (int round = 0; round < 2; ++round) {
      if (todo == 0) break;
      const int lead = __builtin_ctzll(todo);
      const uint32_t v = (uint32_t)__builtin_amdgcn_readlane((int)bkt[it], lead);
      const bool mine = ((todo >> lane) & 1u) && bkt[it] == v;
      const uint64_t mask = __ballot(mine);
      uint32_t at = 0;
      if (lane == (uint32_t)lead) at = atomicAdd(&s_cnt[v], (uint32_t)__popcll(mask));
      if (COUNT && a.e.size) {
        const uint64_t sum = wave::sum<uint64_t>(mine ? sz[it] : 0u);
        if (lane == (uint32_t)lead) atomicAdd(&s_units[v], (unsigned long long)sum);
      }
      if (!COUNT) {
        at = (uint32_t)__builtin_amdgcn_readlane((int)at, lead);
        if (mine) r[it] = at + (uint32_t)__popcll(mask & lanemask_lt);
      }
      todo &= ~mask;
    }
    if ((todo >> lane) & 1u) {
      r[it] = atomicAdd(&s_cnt[bkt[it]], 1u);
      if (COUNT && a.e.size) atomicAdd(&s_units[bkt[it]], (unsigned long long)sz[it]);
    }
  }
  if (COUNT && err) atomicOr((unsigned long long*)a.err, (unsigned long long)err);
  __syncthreads();
  if constexpr (COUNT) {
    if (tid < a.B && s_cnt[tid]) {
      atomicAdd(&a.count[tid], s_cnt[tid]);
      if (a.e.size) atomicAdd((unsigned long long*)&a.units[tid], s_units[tid]);
    }
  } else {
    uint32_t total;
    const uint32_t count = tid < a.B ? a.count[tid] : 0u;
    const uint32_t first = scan_wg(count, s_w, &total);
    if (tid < a.B && s_cnt[tid]) s_base[tid] = first + atomicAdd(&a.taken[tid], s_cnt[tid]);
    if (blockIdx.x == 0) {  // where each bucket begins, for the kernel that sorts them
      __shared__ uint64_t s_w64[BNW];
      uint64_t all;
      const uint64_t below = scan_wg(tid < a.B && a.e.size ? a.units[tid] : (uint64_t)count, s_w64, &all);
      if (tid < a.B) {
        a.first[tid] = first;
        a.below[tid] = below;
        if (count > BUCKET_CAP) *a.over = 1;
      }
      if (tid == 0) {
        a.first[a.B] = total;
        a.below[a.B] = all;
      }
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < IPT; ++it) {
      const uint64_t i = i0 + it * BT;
      if (i >= a.e.N) continue;
      const uint32_t pos = s_base[bkt[it]] + r[it];
      a.key[pos] = la[it];
      a.id[pos] = (uint32_t)i;
    }
  }
}

// Sorts the bucket's n entries (this thread's: key[it], id[it] at it * BT + tid,
// padded to m, a multiple of 64, with entries above every real one) into s_key
// (and s_id unless PACKED): waves sort 64 entries each in registers, then
// sorted lists are merged two by two, each entry finding its place by a binary
// search in the sibling list.
template <bool PACKED>
__device__ inline void sort_bucket(uint64_t (&key)[BUCKET_IPT], uint32_t (&id)[BUCKET_IPT], uint32_t m,
                                   uint64_t* s_key, uint32_t* s_id) {
  const uint32_t tid = threadIdx.x;
  uint32_t to[BUCKET_IPT];
#pragma unroll
  for (int it = 0; it < BUCKET_IPT; ++it) {
    const uint32_t x = it * BT + tid;
    if (x >= m) break;  // whole waves
    sort_wave<PACKED>(key[it], id[it]);
    s_key[x] = key[it];
    if (!PACKED) s_id[x] = id[it];
  }
  __syncthreads();
  for (uint32_t L = 64; L < m; L <<= 1) {
#pragma unroll
    for (int it = 0; it < BUCKET_IPT; ++it) {
      const uint32_t x = it * BT + tid;
      if (x >= m) break;
      key[it] = s_key[x];
      if (!PACKED) id[it] = s_id[x];
      to[it] = merged_place<PACKED>(s_key, s_id, m, L, x, key[it], id[it]);
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < BUCKET_IPT; ++it) {
      const uint32_t x = it * BT + tid;
      if (x >= m) break;
      s_key[to[it]] = key[it];
      if (!PACKED) s_id[to[it]] = id[it];
    }
    __syncthreads();
  }
}

// The least (key, id) with rank[e] of the n entries below it, for two ranks at
// once, in k[e] and i[e]: byte by byte from the top, the byte's value is the one
// that holds the rank among the entries that agree with the bytes found.  A rank
// that reaches zero is done (the bytes left are zero).  Every thread calls it.
__device__ inline void select_ranks(const uint64_t* key, const uint32_t* id, uint32_t n, uint32_t (&rank)[2],
                                    uint64_t (&k)[2], uint32_t (&i)[2], uint32_t (*s_cnt)[256], uint32_t* s_w) {
  __shared__ uint32_t s_byte[2], s_before[2];
  constexpr int ID_BYTES = (BUCKET_ID_BITS + 7) / 8;
  constexpr int U = 2;  // entries per thread whose loads are in flight together
  const uint32_t tid = threadIdx.x;
  const uint64_t lanemask_lt = (1ull << (tid & 63)) - 1ull;
  for (int byte = 8 + ID_BYTES - 1; byte >= 0 && (rank[0] | rank[1]); --byte) {
    const bool in_key = byte >= ID_BYTES;
    const int shift = 8 * (in_key ? byte - ID_BYTES : byte);
    if (tid < 256) s_cnt[0][tid] = s_cnt[1][tid] = 0;
    __syncthreads();
    for (uint32_t x0 = 0; x0 < n; x0 += U * BT) {  // uniform: the ballots need every lane
      uint64_t kx[U];
      uint32_t ix[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const uint32_t x = min(x0 + u * BT + tid, n - 1);
        kx[u] = key[x];
        ix[u] = in_key ? 0u : id[x];
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const bool valid = x0 + u * BT + tid < n;
        const uint32_t d = (in_key ? (uint32_t)(kx[u] >> shift) : ix[u] >> shift) & 255u;
        const uint64_t same = ~wave::digit_differs<8>(d);
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const bool agrees = valid && (in_key ? (kx[u] ^ k[e]) >> shift >> 8 == 0
                                               : kx[u] == k[e] && (ix[u] ^ i[e]) >> shift >> 8 == 0);
          const uint64_t group = same & __ballot(agrees);
          if (agrees && (group & lanemask_lt) == 0) atomicAdd(&s_cnt[e][d], (uint32_t)__popcll(group));
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const uint32_t c = tid < 256 ? s_cnt[e][tid] : 0u;
      uint32_t total;
      const uint32_t before = scan_wg(c, s_w, &total);
      if (before <= rank[e] && rank[e] - before < c) {
        s_byte[e] = tid;
        s_before[e] = before;
      }
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 2; ++e)
      if (rank[e]) {
        rank[e] -= s_before[e];
        if (in_key) k[e] |= (uint64_t)s_byte[e] << shift;
        else i[e] |= s_byte[e] << shift;
      }
    __syncthreads();  // s_byte and s_before are reused
  }
}

// The entries of BUCKET_CAP ranks from r on (or those there are) of a bucket of
// `all` blocks that begins at `first`, in any order, to s_key and s_id; returns
// their number.  *below: size units of the bucket's entries before them, *least:
// no key of theirs is below it.  Every thread calls it.
__device__ inline uint32_t gather_piece(const BucketArgs& a, uint32_t first, uint32_t all, uint32_t r,
                                        uint64_t* below, uint64_t* least, uint64_t* s_key, uint32_t* s_id,
                                        uint64_t* s_w64) {
  __shared__ uint32_t s_cnt[2][256];
  __shared__ uint32_t s_w[BNW];
  __shared__ uint32_t s_taken;
  const uint32_t tid = threadIdx.x;
  const uint32_t n = min(all - r, BUCKET_CAP);
  const bool last = r + n == all;
  uint32_t rank[2] = {r, last ? 0u : r + n};
  uint64_t k[2] = {0, last ? ~0ull : 0ull};
  uint32_t i[2] = {0, last ? ~0u : 0u};
  select_ranks(a.key + first, a.id + first, all, rank, k, i, s_cnt, s_w);
  if (tid == 0) s_taken = 0;
  __syncthreads();
  uint64_t lower = 0;
#pragma unroll 1
  for (uint32_t x = tid; x < all; x += BT) {
    const uint64_t kx = a.key[first + x];
    const uint32_t ix = a.id[first + x];
    if (pair_less(kx, ix, k[0], i[0])) {
      lower += a.e.size ? a.e.size[ix] : 1u;
    } else if (pair_less(kx, ix, k[1], i[1])) {
      const uint32_t at = atomicAdd(&s_taken, 1u);  // below n: those entries are n
      s_key[at] = kx;
      s_id[at] = ix;
    }
  }
  scan_wg(lower, s_w64, below);
  __syncthreads();
  *least = k[0];
  return n;
}

// One bucket per workgroup, sorted in LDS and written out with the prefix.
// Where the bucket's keys span less than 2^44 - 1 (all but the few buckets that
// hold two types, in practice), key and id fit one word below the padding's:
// one compare and two registers an entry instead of three and three (an entry
// equal to the padding would share a place with it in a merge).
//
// A bucket of more than BUCKET_CAP blocks, which only times made to miss the
// sampled blocks leave (none in sweeps of round-robin, strided and contiguous
// layouts), is left to the workgroups past the buckets': each takes BUCKET_CAP
// of its ranks, finds their ends by selection (at most 11 passes over the
// bucket) and sorts the entries between.  With all but the sample in one bucket
// a call takes 0.19-0.28 ms at 20 000 blocks (times distinct - tied), 1.8-2.5 at
// 300 000, 6.1-8.7 at 2^20; ranking every entry against all the others, as
// before, grew with the square.  The idle workgroups cost 0.5 us at 2^20 blocks.
__global__ __launch_bounds__(BT) __attribute__((amdgpu_waves_per_eu(8))) void evict_bucket_kernel(BucketArgs a) {
  __shared__ uint64_t s_key[BUCKET_CAP];
  __shared__ uint32_t s_id[BUCKET_CAP];
  __shared__ uint64_t s_w64[BNW];
  __shared__ uint32_t s_wide;
  const uint32_t tid = threadIdx.x;
  const uint64_t unit = a.e.unit_bytes;
  const uint64_t err = *a.err;
  if (blockIdx.x == 0 && tid == 0) finish_result(a.e, err, a.below[a.B] * unit);
  if (err) return;
  if (tid == 0) s_wide = 0;
  uint32_t first, n;
  uint64_t below, least;  // no key is below `least`
  uint64_t key[BUCKET_IPT];
  uint32_t id[BUCKET_IPT];
  if (blockIdx.x < a.B) {
    first = a.first[blockIdx.x];
    n = a.first[blockIdx.x + 1] - first;
    below = a.below[blockIdx.x];
    least = blockIdx.x ? a.spl_key[blockIdx.x - 1] : 0ull;
    if (n == 0 || n > BUCKET_CAP) return;
#pragma unroll
    for (int it = 0; it < BUCKET_IPT; ++it) {
      const uint32_t x = it * BT + tid;
      if (it * BT >= n) break;  // uniform
      key[it] = x < n ? a.key[first + x] : ~0ull;
      id[it] = x < n ? a.id[first + x] : ~0u;
    }
  } else {
    if (!*a.over) return;
    uint32_t b = 0, r = 0, piece = a.B;  // piece: the workgroup of ranks r.. of bucket b
    for (; b < a.B; ++b) {
      const uint32_t all = a.first[b + 1] - a.first[b];
      if (all <= BUCKET_CAP) continue;
      r = (blockIdx.x - piece) * BUCKET_CAP;
      if (r < all) break;
      piece += (all + BUCKET_CAP - 1) / BUCKET_CAP;
    }
    if (b == a.B) return;
    first = a.first[b];
    n = gather_piece(a, first, a.first[b + 1] - first, r, &below, &least, s_key, s_id, s_w64);
    first += r;
    below += a.below[b];
#pragma unroll
    for (int it = 0; it < BUCKET_IPT; ++it) {
      const uint32_t x = it * BT + tid;
      if (it * BT >= n) break;  // uniform
      key[it] = x < n ? s_key[x] : ~0ull;
      id[it] = x < n ? s_id[x] : ~0u;
    }
  }
  const uint32_t m = (n + 63) & ~63u;
  bool wide = false;
#pragma unroll
  for (int it = 0; it < BUCKET_IPT; ++it)
    wide |= it * BT + tid < n && ((key[it] - least + 1) >> (64 - BUCKET_ID_BITS)) != 0;
  __syncthreads();  // s_wide is zero
  if (wide) s_wide = 1;
  __syncthreads();
  const bool packed = !s_wide;
  if (packed) {
#pragma unroll
    for (int it = 0; it < BUCKET_IPT; ++it) {
      const uint32_t x = it * BT + tid;
      if (x >= m) break;
      if (x < n) key[it] = ((key[it] - least) << BUCKET_ID_BITS) | id[it];
    }
    sort_bucket<true>(key, id, m, s_key, s_id);
  } else {
    sort_bucket<false>(key, id, m, s_key, s_id);
  }
#pragma unroll
  for (int it = 0; it < BUCKET_IPT; ++it) {
    if (it * BT >= n) break;  // uniform
    const uint32_t x = it * BT + tid;
    const uint32_t b = x >= n ? 0u : packed ? (uint32_t)s_key[x] & ((1u << BUCKET_ID_BITS) - 1) : s_id[x];
    const uint64_t own = x >= n ? 0ull : a.e.size ? a.e.size[b] : 1ull;
    uint64_t sum;
    const uint64_t ex = scan_wg(own, s_w64, &sum);
    if (x < n) emit(a.e, first + x, b, (below + ex + own) * unit, own * unit);
    below += sum;
  }
}

void launch_buckets(const EvictArgs& e, uint8_t* w, hipStream_t s) {
  const uint32_t N = e.N;
  BucketArgs a{};
  a.e = e;
  a.B = bucket_count(N);
  a.S = sample_count(a.B);
  const BucketLayout l = bucket_layout(N);
  a.key = reinterpret_cast<uint64_t*>(w + l.key);
  a.id = reinterpret_cast<uint32_t*>(w + l.id);
  a.spl_key = reinterpret_cast<uint64_t*>(w + l.spl_key);
  a.units = reinterpret_cast<uint64_t*>(w + l.units);
  a.spl_id = reinterpret_cast<uint32_t*>(w + l.spl_id);
  a.count = reinterpret_cast<uint32_t*>(w + l.count);
  a.taken = reinterpret_cast<uint32_t*>(w + l.taken);
  a.first = reinterpret_cast<uint32_t*>(w + l.first);
  a.below = reinterpret_cast<uint64_t*>(w + l.below);
  a.over = reinterpret_cast<uint32_t*>(w + l.over);
  a.sample = reinterpret_cast<uint64_t*>(w + l.sample);
  a.err = reinterpret_cast<uint64_t*>(w + l.err);
  if (a.S <= DIRECT_WG * BNW) {
    hipLaunchKernelGGL((evict_splitter_kernel<1, false>), dim3(DIRECT_WG), dim3(BT), 0, s, a);
  } else {
    hipLaunchKernelGGL(evict_sample_kernel, dim3((a.S + SAMPLE_WG - 1) / SAMPLE_WG), dim3(SAMPLE_WG), 0, s, a);
    hipLaunchKernelGGL((evict_splitter_kernel<2, true>), dim3(DIRECT_WG), dim3(BT), 0, s, a);
  }
  if (N <= PARTITION_ONE_MAX) {
    const dim3 grid((N + BT - 1) / BT);
    hipLaunchKernelGGL((evict_partition_kernel<1, true>), grid, dim3(BT), 0, s, a);
    hipLaunchKernelGGL((evict_partition_kernel<1, false>), grid, dim3(BT), 0, s, a);
  } else {
    const dim3 grid((N + 2 * BT - 1) / (2 * BT));
    hipLaunchKernelGGL((evict_partition_kernel<2, true>), grid, dim3(BT), 0, s, a);
    hipLaunchKernelGGL((evict_partition_kernel<2, false>), grid, dim3(BT), 0, s, a);
  }
  // a bucket of n > BUCKET_CAP blocks has at most 2 n / BUCKET_CAP pieces
  hipLaunchKernelGGL(evict_bucket_kernel, dim3(a.B + N / (BUCKET_CAP / 2)), dim3(BT), 0, s, a);
}

void launch_radix(EvictArgs& a, uint8_t* w, hipStream_t s) {
  const RadixLayout l = radix_layout(a.N);
  a.ntiles = radix_tiles(a.N);
  for (int i = 0; i < 2; ++i) {
    a.keys[i] = reinterpret_cast<uint64_t*>(w + l.keys[i]);
    a.vals[i] = reinterpret_cast<uint32_t*>(w + l.vals[i]);
  }
  a.hist = reinterpret_cast<uint32_t*>(w + l.hist);
  a.dtot = reinterpret_cast<uint32_t*>(w + l.dtot);
  a.tile_sum = reinterpret_cast<uint64_t*>(w + l.tile_sum);
  if (!a.prefix) a.prefix = reinterpret_cast<uint64_t*>(w + l.prefix);
  a.misc = reinterpret_cast<uint64_t*>(w + l.misc);
  hipLaunchKernelGGL(evict_init_kernel, dim3(1), dim3(1), 0, s, a);
  hipLaunchKernelGGL(evict_keys_kernel, dim3(a.ntiles < KEY_WG_MAX ? a.ntiles : KEY_WG_MAX), dim3(ET), 0, s, a);
  for (int shift = 0; shift < 64; shift += 8) {
    hipLaunchKernelGGL(evict_hist_kernel, dim3(a.ntiles), dim3(ET), 0, s, a, shift);
    hipLaunchKernelGGL(evict_dscan_kernel, dim3(256), dim3(ET), 0, s, a, shift);
    hipLaunchKernelGGL(evict_scatter_kernel, dim3(a.ntiles), dim3(ET), 0, s, a, shift);
  }
  hipLaunchKernelGGL(evict_prefix_tiles_kernel, dim3(a.ntiles), dim3(ET), 0, s, a);
  if (a.ntiles <= FIX_SCAN_TILES) {
    hipLaunchKernelGGL(evict_prefix_fix_scan_kernel, dim3(a.ntiles), dim3(ET), 0, s, a);
  } else {
    hipLaunchKernelGGL(evict_prefix_top_kernel, dim3(1), dim3(1024), 0, s, a);
    hipLaunchKernelGGL(evict_prefix_fix_kernel, dim3(a.ntiles), dim3(ET), 0, s, a);
    hipLaunchKernelGGL(evict_result_kernel, dim3(1), dim3(1), 0, s, a);
  }
}

}  // namespace

hipError_t launch_evict(uint32_t N, const uint8_t* type, const uint64_t* last_access, const uint32_t* size,
                        uint64_t unit_bytes, uint32_t tier, uint64_t need, void* workspace, uint32_t* order,
                        uint64_t* prefix, uint32_t* result, hipStream_t s) {
  EvictArgs a{};
  a.N = N;
  a.tier = tier;
  a.type = type;
  a.last_access = last_access;
  a.size = size;
  a.unit_bytes = unit_bytes;
  a.need = need;
  a.order = order;
  a.prefix = prefix;
  a.result = result;
  uint8_t* w = static_cast<uint8_t*>(workspace);
  if (N <= DIRECT_MAX) launch_direct(a, s);
  else if (N <= BUCKET_MAX) launch_buckets(a, w, s);
  else launch_radix(a, w, s);
  return hipGetLastError();
}

}  // namespace mori
