// Rank / boundary step of one rebalance: the placement in a single workgroup.
//
//   1. idleness of every program by Eq. 1 (Sec. 4.2), binary32, totals
//      accumulated oldest cycle first from +0, correctly rounded division;
//   2. a 64-bit key per program and a stable sort of (key, id): sorted waves
//      merged two by two, or for many programs or long windows ranks counted
//      by two kernels before this one.  Boundary policy: the key is the idleness bits,
//      optionally with the Acting bit of the demotion order of Sec. 4.3.1 --
//      the relative ranking, busiest first.  Incremental policy (Sec. 4.3.1):
//      the key is the program's listing group (old tier; Waiting split into
//      returning, new and Acting) above its priority in that group, so each
//      tier group lists its programs in reverse demotion order and the
//      promotion candidates come in promotion order;
//   3. an inclusive u64 scan of KV bytes in that order, then either the two
//      capacity boundaries (Sec. 4.1 per-tier capacity, Sec. 7.2 fill from the
//      busiest end) or the greedy skip-fit walk, or the incremental policy:
//      demote-until-fits is the tail of a tier group past its longest fitting
//      prefix, promote-while-fits a prefix of the candidates' byte scan;
//      victims that do not all fit the CPU room, skip-fit promotion and the
//      skip-fit walk go 64 at a time by one wave;
//   4. the sticky diff (Sec. 4.3): per-program transition category, the
//      swap-out and swap-in lists in that order and the page/slot bases.
//
// P <= 4096 programs fit in LDS (4 per thread), so placement and diff are one
// launch, for up to 1024 programs with windows of up to 2^14 cycles in all the
// whole step (5 us for tens of programs, 7 for 256), bound by the one workgroup's
// vector ALU and barriers; nothing here is bandwidth-bound.
#include "mori_internal.h"
#include "sort.h"
#include "wave.h"

namespace mori {
namespace {

// Four shapes, chosen by P at launch: one wave (64 threads, so every barrier
// is a single wave's) for P <= 64, 256 threads x 1 item up to 256, 1024 x 1 up
// to 1024 and 1024 threads x 4 items (striped: item x = it * RT + tid) up to
// 4096.  The one workgroup computes and sorts the keys of up to
// SORT_MAX_PROGRAMS programs itself; above, and where the windows together hold
// more than SORT_MAX_CYCLES cycles, two kernels before it do that on many
// compute units.  Those cost about 4.5 us a plan; the one workgroup took 13 us
// to sort 4096 programs in radix passes (merging them was not built: 54 LDS
// gathers for each of 64 waves, at about 10 clocks, come to 14 us) and takes
// 0.5 ns for each cycle it reads.  A pair of plans,
// sorted -> counted: 4096 programs with 5 cycles each 112 -> 100 us, with 64
// 380 -> 108; 1100 programs 92 -> 81 and 150 -> 86; 1024 programs with 5 stay
// at 72, with 64 go from 134 to 85, 300 with 64 stay at 82.
constexpr uint32_t SORT_MAX_PROGRAMS = 1024, SORT_MAX_CYCLES = 1u << 14;
constexpr int ID_BITS = 12;      // a program id
constexpr int GROUP_SHIFT = 61;  // incremental keys: listing group in the top three bits
constexpr uint64_t ACTING_BIT = 0x80000000u;  // ... and statuses in the key, above the idleness bits
constexpr int KEY_WG = 64, RANK_WG = 1024;

// Exclusive scans of the IPT x RT items in rank order (item it of thread tid
// has rank it * RT + tid), N values per item side by side: wave scans, the
// per-(slice, wave) totals scanned by the first wave, and three barriers in
// all, however many slices.  Blocks and programs, whose totals a table's 32-bit
// offsets bound: a 32-bit step is one instruction where a 64-bit one is four.
// s_tot needs (IPT * NW + 1) * N entries; total[n] receives the sum of value n
// over all items.
template <int NW, int IPT, int N>
__device__ void scan_slices(const uint32_t (&v)[IPT][N], uint32_t (&ex)[IPT][N], uint32_t* s_tot,
                            uint32_t (&total)[N]) {
  constexpr int NS = IPT * NW;
  static_assert(NS <= 64, "one lane per (slice, wave) total");
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
  for (int it = 0; it < IPT; ++it)
#pragma unroll
    for (int n = 0; n < N; ++n) {
      const uint32_t x = wave::incl_add(v[it][n]);
      ex[it][n] = x - v[it][n];
      if (lane == 63) s_tot[(it * NW + wid) * N + n] = x;
    }
  __syncthreads();
  if (wid == 0) {
#pragma unroll
    for (int n = 0; n < N; ++n) {
      const uint32_t w = lane < NS ? s_tot[lane * N + n] : 0u;
      const uint32_t wi = wave::incl_add(w);
      if (lane < NS) s_tot[lane * N + n] = wi - w;
      if (lane == NS - 1) s_tot[NS * N + n] = wi;
    }
  }
  __syncthreads();
#pragma unroll
  for (int it = 0; it < IPT; ++it)
#pragma unroll
    for (int n = 0; n < N; ++n) ex[it][n] += s_tot[(it * NW + wid) * N + n];
#pragma unroll
  for (int n = 0; n < N; ++n) total[n] = s_tot[NS * N + n];
  __syncthreads();
}

// Adds every thread's v into an LDS total with one atomic per wavefront (the
// wave's sum by DPP); every thread of the workgroup calls it.
__device__ inline void add_to(uint32_t* dst, uint32_t v) {
  const uint32_t t = wave::sum(v);
  if ((threadIdx.x & 63) == 0 && t) atomicAdd(dst, t);
}
// Largest p in [0, P) with off[p] <= e (so off[p] <= e < off[p+1] when e < off[P]).
__device__ inline uint32_t find_program(const uint32_t* off, uint32_t P, uint32_t e) {
  uint32_t lo = 0, hi = P;  // invariant: off[lo] <= e, answer in [lo, hi)
  while (hi - lo > 1) {
    const uint32_t mid = (lo + hi) >> 1;
    if (off[mid] <= e) lo = mid;
    else hi = mid;
  }
  return lo;
}

// Owner of every page, from the block tables alone (the placement is not known
// yet), and the ownership errors: a page owned twice, owned and free or out of
// range, a page held by a CPU/Waiting program.  Workgroup b of nb.  The program
// data is validated by the ranking workgroup at the same time, so nothing here
// relies on it: entries are bounded by the table, programs by P.
__device__ void claim_pages(const PlanArgs& a, uint32_t b, uint32_t nb) {
  if (a.P == 0) return;
  const uint32_t used = min(a.tbl_off[a.P], a.tbl_len);
  uint32_t err = 0;
  for (uint64_t e64 = (uint64_t)b * blockDim.x + threadIdx.x; e64 < used; e64 += (uint64_t)nb * blockDim.x) {
    const uint32_t e = (uint32_t)e64;  // 64-bit stride: no wrap near 2^32 entries
    const uint32_t pg = a.tbl[e];
    const uint32_t p = find_program(a.tbl_off, a.P, e);
    if (a.tier[p] != MORI_TIER_GPU) {
      if (pg != MORI_NO_PAGE) err |= MORI_DEV_NONRES_PAGE;
      continue;
    }
    if (pg >= a.NB) {
      err |= MORI_DEV_PAGE_RANGE;
      continue;
    }
    const unsigned long long mine = ((unsigned long long)p << 32) | (e + 1u);
    if (atomicExch((unsigned long long*)&a.owner[pg], mine) != 0 || a.free_map[pg]) err |= MORI_DEV_PAGE_DUP;
  }
  if (err) atomicOr(a.page_err, err);
}

// A program's key and blocks (Eq. 1 or the idleness given); what is wrong with
// its data goes to err.  Every load of the program first, none behind a branch,
// so they are in flight together: one memory latency instead of one per load.
__device__ inline uint64_t program_key(const PlanArgs& a, uint32_t x, uint8_t& told, uint32_t& blocks, uint32_t& err) {
  const bool given = (a.flags & MORI_F_IDLENESS_GIVEN) != 0;
  const bool incremental = (a.flags & MORI_F_INCREMENTAL) != 0;
  const bool need_status = incremental || (a.flags & MORI_F_STATUS_KEY);
  told = a.tier[x];
  const uint32_t off0 = a.tbl_off[x], off1 = a.tbl_off[x + 1];
  const uint8_t st = need_status ? a.status[x] : 0;
  float rv[8], cv[8];  // the first eight cycles of the window
  const float* w = given ? nullptr : a.window + (size_t)x * a.k * 2;
  if (!given) {
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      if ((uint32_t)u >= a.k) break;  // uniform
      rv[u] = w[2 * u];
      cv[u] = w[2 * u + 1];
    }
  }
  if (told > ((a.flags & MORI_F_SSD_TIER) ? MORI_TIER_SSD : MORI_TIER_WAIT)) err |= MORI_DEV_BAD_TIER;
  if (off1 < off0) err |= MORI_DEV_BAD_TBL_OFF;
  blocks = off1 - off0;
  float v;
  if (given) {
    v = a.idleness[x];
    if (!(v >= 0.0f && v <= 1.0f)) err |= MORI_DEV_BAD_IDLENESS;
  } else {
    float t_reasoning = 0.0f, t_acting = 0.0f;
    for (uint32_t j0 = 0; j0 < a.k; j0 += 8) {  // eight cycles' loads in flight, then the sums in order
      if (j0 > 0) {
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const uint32_t j = min(j0 + u, a.k - 1);
          rv[u] = w[2 * j];
          cv[u] = w[2 * j + 1];
        }
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        if (j0 + u >= a.k) break;
        const float r = rv[u], c = cv[u];
        if (!(r >= 0.0f) || !(c >= 0.0f) || __builtin_isinf(r) || __builtin_isinf(c)) err |= MORI_DEV_BAD_WINDOW;
        t_reasoning = t_reasoning + r;
        t_acting = t_acting + c;
      }
    }
    const float total = t_reasoning + t_acting;
    if (__builtin_isinf(t_reasoning) || __builtin_isinf(t_acting) || __builtin_isinf(total)) err |= MORI_DEV_BAD_WINDOW;
    v = (total > 0.0f) ? t_acting / total : 0.0f;
  }
  if (v == 0.0f) v = 0.0f;  // a negative zero keys like +0
  const uint32_t bits = __float_as_uint(v);  // < 2^30 for idleness in [0, 1]
  if (!incremental) {
    uint64_t k = bits;
    if ((a.flags & MORI_F_STATUS_KEY) && st == MORI_ST_ACTING) k |= ACTING_BIT;
    return k;
  }
  if (st > MORI_ST_NEW) err |= MORI_DEV_BAD_STATUS;
  const uint64_t acting = st == MORI_ST_ACTING;
  uint64_t grp;
  uint64_t sub = bits;
  if (told == MORI_TIER_GPU || told == MORI_TIER_CPU) {
    grp = told;  // Reasoning before Acting, then idleness: the reverse of the demotion order
    if (acting) sub |= ACTING_BIT;
  } else if (st == MORI_ST_NEW) {
    grp = 3;  // new arrivals: smallest context first
    if (blocks >= 0x80000000u) err |= MORI_DEV_BAD_TBL_OFF;
    sub |= (uint64_t)blocks << 30;
  } else {
    grp = acting ? 4 : 2;
  }
  return (grp << GROUP_SHIFT) | sub;
}

// The table's ends.  One thread.
__device__ inline uint32_t table_error(const PlanArgs& a) {
  return a.tbl_off[0] != 0u || a.tbl_off[a.P] > a.tbl_len ? MORI_DEV_BAD_TBL_OFF : 0u;
}

// ---- more than one workgroup sorts well: keys and ranks by many -----------
// Keys, one program a thread in workgroups of a wave, so that the windows are
// read by many compute units.
__global__ __launch_bounds__(KEY_WG) void program_keys_kernel(PlanArgs a) {
  const uint32_t x = blockIdx.x * KEY_WG + threadIdx.x;
  uint32_t err = 0, blocks;
  uint8_t told;
  if (x == 0) err |= table_error(a);
  if (x < a.P) a.key[x] = program_key(a, x, told, blocks, err);
  err = wave::all_or<uint32_t>(err);
  if (threadIdx.x == 0) a.key_err[blockIdx.x] = err;
}

// Ranks, one program a wave: the programs before it are counted.  Keys of
// rejected programs are ranked like any others (the order is total whatever
// they hold); the placement reports the error.  What it reads of a program goes
// to the program's rank: id | listing group << 16 | Acting bit << 20 |
// blocks << 32.
__global__ __launch_bounds__(RANK_WG) void program_rank_kernel(PlanArgs a) {
  __shared__ uint64_t s_key[MORI_MAX_PROGRAMS];
  const uint32_t chunks = (a.P + 64 * GROUP - 1) / (64 * GROUP) * GROUP;
  const uint32_t p = blockIdx.x * (RANK_WG / 64) + (threadIdx.x >> 6);
  const uint32_t own = min(p, a.P - 1);
  const uint32_t off0 = a.tbl_off[own], off1 = a.tbl_off[own + 1];
  for (uint32_t j = threadIdx.x; j < chunks * 64; j += RANK_WG) s_key[j] = j < a.P ? a.key[j] : ~0ull;
  __syncthreads();
  if (p >= a.P) return;
  uint32_t rank[1];
  uint64_t unused[1];
  count_before<1, false>(s_key, nullptr, chunks, p, rank, unused);
  if ((threadIdx.x & 63) == 0) {
    const uint64_t k = s_key[p];
    a.rank_rec[rank[0]] = p | ((k >> GROUP_SHIFT) << 16) | ((k & ACTING_BIT) ? 1ull << 20 : 0ull) |
                          ((uint64_t)(off1 - off0) << 32);
  }
}

// Sorts one (key, id) per thread, padded above P programs: entries 0 .. P - 1
// (and the padding to a multiple of 64) end up ascending in s_key (and s_id
// unless PACKED).
template <bool PACKED>
__device__ void sort_programs(uint64_t key, uint32_t id, uint32_t P, uint64_t* s_key, uint32_t* s_id) {
  const uint32_t m = (P + 63) & ~63u;
  const uint32_t x = threadIdx.x;
  const bool active = x < m;  // whole waves
  if (active) {
    sort_wave<PACKED>(key, id, P);
    s_key[x] = key;
    if (!PACKED) s_id[x] = id;
  }
  __syncthreads();
  for (uint32_t L = 64; L < m; L <<= 1) {
    uint32_t to = 0;
    if (active) {
      key = s_key[x];
      if (!PACKED) id = s_id[x];
      to = merged_place<PACKED>(s_key, s_id, m, L, x, key, id);
    }
    __syncthreads();
    if (active) {
      s_key[to] = key;
      if (!PACKED) s_id[to] = id;
    }
    __syncthreads();
  }
}

// Skip-fit over 64 candidates in lane order: each is taken if it still fits the
// room left when its turn comes.  b: this lane's blocks; pending: the
// candidates; returns those taken and lowers room (blocks).  A round takes the
// longest run that fits together: the candidate after it, and any that is
// larger than the room left, can never be taken.  All lanes call it.
__device__ inline uint64_t take_fitting(uint64_t pending, uint64_t b, uint64_t& room) {
  const uint32_t lane = threadIdx.x & 63;
  uint64_t taken = 0;
  for (;;) {
    pending &= __ballot(b <= room);
    if (!pending) return taken;
    const uint64_t sum = wave::incl_add<uint64_t>((pending >> lane) & 1u ? b : 0u);
    const uint64_t fits = pending & __ballot(sum <= room);  // a run: the sums never decrease, and the first one fits
    room -= wave::lane_of(sum, 63 - __builtin_clzll(fits));
    taken |= fits;
    pending &= ~fits;
  }
}

// Skip-fit over ranks [lo, hi) (in reverse: hi - 1 down to lo) by one wave:
// those taken go to `tier`.  One thread over the ranks took 0.1 us a program
// (incremental skip-fit, 1024 programs 7.2 us).
template <bool REVERSE>
__device__ void walk_fit(const uint32_t* blocks, uint8_t* tiers, uint32_t lo, uint32_t hi, uint64_t& room,
                         uint8_t tier) {
  const uint32_t lane = threadIdx.x & 63;
  for (uint32_t c = lo; c < hi; c += 64) {
    const bool valid = c + lane < hi;
    const uint32_t r = REVERSE ? hi - 1 - (c - lo + lane) : c + lane;
    const uint64_t taken = take_fitting(__ballot(valid), valid ? blocks[r] : 0u, room);
    if ((taken >> lane) & 1u) tiers[r] = tier;
  }
}

// Transition category.  Leaving the GPU for a tier that keeps the KV (CPU,
// SSD) is a swap-out, the reverse a swap-in.
__device__ inline uint8_t category(uint8_t from, uint8_t to) {
  if (from == to) return MORI_CAT_KEPT;
  switch (from) {
    case MORI_TIER_GPU: return to == MORI_TIER_WAIT ? MORI_CAT_DROP_GPU : MORI_CAT_OUT;
    case MORI_TIER_CPU:
      return to == MORI_TIER_GPU ? MORI_CAT_IN : (to == MORI_TIER_SSD ? MORI_CAT_CPU_SSD : MORI_CAT_DROP_CPU);
    case MORI_TIER_SSD:
      return to == MORI_TIER_GPU ? MORI_CAT_IN : (to == MORI_TIER_CPU ? MORI_CAT_SSD_CPU : MORI_CAT_DROP_SSD);
    default:
      return to == MORI_TIER_GPU ? MORI_CAT_ADMIT_GPU : (to == MORI_TIER_CPU ? MORI_CAT_ADMIT_CPU : MORI_CAT_ADMIT_SSD);
  }
}

// RANKED: program_rank_kernel has ranked the programs.
template <int RT, int IPT, bool RANKED>
__global__ __launch_bounds__(RT) void rank_partition_kernel(PlanArgs a) {
  constexpr int NW = RT / 64;  // wavefronts
  static_assert(RANKED || IPT == 1, "one program a thread is sorted");
  __shared__ uint64_t s_key[RT * IPT];  // sort scratch, then the inclusive byte prefix by rank
  __shared__ uint32_t s_id[RT * IPT];   // sort scratch, then blocks by rank
  __shared__ uint8_t s_tier[RT * IPT];
  __shared__ uint32_t s_nblk[RT * IPT];  // blocks of program x, then its page base
  __shared__ uint8_t s_told[RT * IPT];   // old tier of program x
  __shared__ uint32_t s_tot[(IPT * NW + 1) * 5];
  __shared__ unsigned long long s_or;
  __shared__ uint32_t s_err, s_m_gpu, s_m_cpu, s_m_ssd;
  __shared__ uint32_t s_grp[5], s_cpu_reasoning, s_k_gpu, s_k_cpu;
  __shared__ uint32_t s_n_drop, s_n_admit_cpu, s_gpu_after, s_cpu_after, s_ssd_after;
  __shared__ unsigned long long s_gpu_part, s_upper_part;

  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  if (blockIdx.x > 0) {  // the other workgroups find the pages' owners meanwhile
    claim_pages(a, blockIdx.x - 1, gridDim.x - 1);
    return;
  }
  const uint32_t P = a.P;
  const bool incremental = (a.flags & MORI_F_INCREMENTAL) != 0;
  const bool ssd = (a.flags & MORI_F_SSD_TIER) != 0;
  if (tid == 0) {
    s_err = 0;
    s_or = 0;
    s_m_gpu = s_m_cpu = s_m_ssd = 0;
    for (int g = 0; g < 5; ++g) s_grp[g] = 0;
    s_cpu_reasoning = s_k_gpu = s_k_cpu = 0;
    s_n_drop = s_n_admit_cpu = 0;
    s_gpu_after = s_cpu_after = s_ssd_after = 0;
    s_gpu_part = s_upper_part = 0;
  }
  __syncthreads();

  // ---- 1. validation, Eq. 1, keys --------------------------------------
  uint64_t key[IPT];
  uint32_t id[IPT];
  uint32_t err = 0;
  uint32_t grp[IPT];    // incremental: listing group
  bool acting[IPT];     // ... and Acting
  uint32_t nb[IPT];
  unsigned long long k_or = 0;
  if constexpr (RANKED) {
    if ((uint32_t)tid < (P + KEY_WG - 1) / KEY_WG) err = a.key_err[tid];
#pragma unroll
    for (int it = 0; it < IPT; ++it) {
      const uint32_t r = it * RT + tid;
      const uint64_t rec = r < P ? a.rank_rec[r] : 0ull;
      if (r < P) s_told[r] = a.tier[r];
      id[it] = (uint32_t)rec & ((1u << ID_BITS) - 1u);
      grp[it] = (uint32_t)(rec >> 16) & 7u;
      acting[it] = ((rec >> 20) & 1u) != 0;
      nb[it] = (uint32_t)(rec >> 32);
    }
  } else {
    if (tid == 0) err |= table_error(a);
    key[0] = ~0ull;  // padding sorts after every real key
    id[0] = tid;
    if ((uint32_t)tid < P) k_or = key[0] = program_key(a, tid, s_told[tid], s_nblk[tid], err);
    const uint64_t w_or = wave::all_or<uint64_t>(k_or);
    if (lane == 0 && w_or) atomicOr(&s_or, (unsigned long long)w_or);
  }
  if (err) atomicOr(&s_err, err);
  __syncthreads();
  if (s_err) {
    if (tid == 0) {
      DevSummary z = {};
      z.num_programs = P;
      z.error = s_err;
      *a.sum = z;
      *host_mirror(a, a.sum) = z;
      a.swap_err[0] = a.swap_err[1] = 0;
    }
    return;
  }

  // ---- 2. stable sort of (key, id) ---------------------------------------
  if constexpr (!RANKED) {
    // Incremental keys: the listing group moves down from the top bits to just
    // above the highest bit any program's priority uses (the same order), which
    // mostly leaves room for the id.
    uint32_t gshift = GROUP_SHIFT;
    uint64_t kor = s_or;
    if (incremental) {
      constexpr uint64_t SUB = (1ull << GROUP_SHIFT) - 1;
      const uint64_t sub_or = kor & SUB;
      gshift = sub_or ? 64u - (uint32_t)__clzll(sub_or) : 0u;
      auto pack = [&](uint64_t k) { return ((k >> GROUP_SHIFT) << gshift) | (k & SUB); };
      if ((uint32_t)tid < P) key[0] = pack(key[0]);
      kor = pack(kor);
    }
    // One program a thread, waves sorted and lists merged in LDS.  Boundary
    // keys, and incremental ones of less than 2^20 blocks, leave room for the
    // id in the same word.  (Counting ranks against keys in LDS took 7.1 us at
    // 256 programs, radix passes 5.2 us at 1024 and 7.6 us with incremental
    // keys; this 2.0 and 4.3 us.)
    const uint32_t x = tid;
    if ((kor >> (64 - ID_BITS)) == 0) {
      sort_programs<true>(x < P ? (key[0] << ID_BITS) | x : ~0ull, x, P, s_key, s_id);
      key[0] = s_key[tid] >> ID_BITS;
      id[0] = (uint32_t)s_key[tid] & ((1u << ID_BITS) - 1u);
    } else {
      sort_programs<false>(key[0], id[0], P, s_key, s_id);
      key[0] = s_key[tid];
      id[0] = s_id[tid];
    }
    grp[0] = (uint32_t)(key[0] >> gshift);
    acting[0] = gshift && (key[0] & ((1ull << gshift) - 1) & ACTING_BIT);
    nb[0] = x < P ? s_nblk[id[0]] : 0u;
    __syncthreads();  // s_key and s_id are reused
  }
  // item x now holds rank x: id[it] is the program at rank it * RT + tid
#pragma unroll
  for (int it = 0; it < IPT; ++it) s_id[it * RT + tid] = nb[it];

  // ---- 3. KV-byte prefix in that order and the placement ----------------
  uint64_t S[IPT];
  {
    uint32_t blocks[IPT][1], ex[IPT][1], tot[1];
#pragma unroll
    for (int it = 0; it < IPT; ++it) blocks[it][0] = nb[it];
    scan_slices<NW, IPT, 1>(blocks, ex, s_tot, tot);
#pragma unroll
    for (int it = 0; it < IPT; ++it) {
      S[it] = (uint64_t)(ex[it][0] + nb[it]) * a.block_bytes;
      s_key[it * RT + tid] = S[it];
    }
  }
  if (incremental) {
    // listing groups: [0, g1) GPU, [g1, g2) CPU, [g2, g3) Waiting returning,
    // [g3, g4) new arrivals, [g4, P) Waiting Acting
    uint32_t gc[5] = {0, 0, 0, 0, 0}, cr = 0;
#pragma unroll
    for (int it = 0; it < IPT; ++it) {
      const uint32_t r = it * RT + tid;
      const uint32_t g = r < P ? grp[it] : 5u;
#pragma unroll
      for (int j = 0; j < 5; ++j) gc[j] += g == (uint32_t)j;
      cr += g == MORI_TIER_CPU && !acting[it];
    }
#pragma unroll
    for (int j = 0; j < 5; ++j) add_to(&s_grp[j], gc[j]);
    add_to(&s_cpu_reasoning, cr);
    __syncthreads();
    const uint32_t g1 = s_grp[0], g2 = g1 + s_grp[1], g3 = g2 + s_grp[2], g4 = g3 + s_grp[3];
    const uint64_t gpu_total = g1 ? s_key[g1 - 1] : 0;
    // (1) CPU admission control and (2) demotion from GPU: each tier keeps the
    // longest prefix of its group that fits its budget (the rest, in reverse,
    // is the demotion order's shortest prefix whose removal fits)
    uint32_t kg = 0, kc = 0;
#pragma unroll
    for (int it = 0; it < IPT; ++it) {
      const uint32_t r = it * RT + tid;
      if (r < g1 && S[it] <= a.gpu_bytes) ++kg;
      if (r >= g1 && r < g2 && S[it] - gpu_total <= a.cpu_bytes) ++kc;
    }
    add_to(&s_k_gpu, kg);
    add_to(&s_k_cpu, kc);
    __syncthreads();
    const uint32_t k_gpu = s_k_gpu, k_cpu = s_k_cpu;
    const uint64_t gpu_kept = k_gpu ? s_key[k_gpu - 1] : 0;
    const uint64_t cpu_kept = k_cpu ? s_key[g1 + k_cpu - 1] - gpu_total : 0;
    const uint64_t room_cpu = a.cpu_bytes - cpu_kept;
    const uint64_t room_gpu = a.gpu_bytes - gpu_kept;
    const bool victims_fit = gpu_total - gpu_kept <= room_cpu;
    const uint32_t c_end = g1 + min(k_cpu, s_cpu_reasoning);  // CPU candidates: [g1, c_end)
#pragma unroll
    for (int it = 0; it < IPT; ++it) {
      const uint32_t r = it * RT + tid;
      uint8_t t;
      if (r < k_gpu) t = MORI_TIER_GPU;
      else if (r < g1) t = victims_fit ? MORI_TIER_CPU : MORI_TIER_WAIT;  // else walked below
      else if (r < g1 + k_cpu) t = MORI_TIER_CPU;
      else t = MORI_TIER_WAIT;
      s_tier[r] = t;
    }
    // (3) promotion: a strict prefix of the candidates' byte scan
    if (!(a.flags & MORI_F_SKIP_FIT)) {
      uint32_t cb[IPT][1], ex[IPT][1], tot[1];
      bool cand[IPT];
#pragma unroll
      for (int it = 0; it < IPT; ++it) {
        const uint32_t r = it * RT + tid;
        cand[it] = (r >= g1 && r < c_end) || (r >= g2 && r < g4);
        cb[it][0] = cand[it] ? nb[it] : 0u;
      }
      scan_slices<NW, IPT, 1>(cb, ex, s_tot, tot);
#pragma unroll
      for (int it = 0; it < IPT; ++it)
        if (cand[it] && (uint64_t)(ex[it][0] + cb[it][0]) * a.block_bytes <= room_gpu) s_tier[it * RT + tid] = MORI_TIER_GPU;
    }
    __syncthreads();
    if (wid == 0) {
      // each victim, most demotable first, to the CPU tier if it still fits
      if (!victims_fit) {
        uint64_t room = room_cpu / a.block_bytes;
        walk_fit<true>(s_id, s_tier, k_gpu, g1, room, MORI_TIER_CPU);
      }
      if (a.flags & MORI_F_SKIP_FIT) {
        // the returning programs and new arrivals go on with the room the CPU programs left
        uint64_t room = room_gpu / a.block_bytes;
        walk_fit<false>(s_id, s_tier, g1, c_end, room, MORI_TIER_GPU);
        walk_fit<false>(s_id, s_tier, g2, g4, room, MORI_TIER_GPU);
      }
    }
    __syncthreads();
    uint32_t ng = 0, nc = 0;
#pragma unroll
    for (int it = 0; it < IPT; ++it) {
      const uint32_t r = it * RT + tid;
      if (r >= P) continue;
      ng += s_tier[r] == MORI_TIER_GPU;
      nc += s_tier[r] == MORI_TIER_CPU;
    }
    add_to(&s_m_gpu, ng);
    add_to(&s_m_cpu, nc);
  } else if (!(a.flags & MORI_F_SKIP_FIT)) {
    // S is non-decreasing in rank order, so the longest feasible prefix is
    // the number of ranks whose inclusive prefix fits the budget.
    uint32_t c = 0;
#pragma unroll
    for (int it = 0; it < IPT; ++it)
      if (it * RT + tid < (int)P && S[it] <= a.gpu_bytes) ++c;
    add_to(&s_m_gpu, c);
    __syncthreads();
    const uint32_t m_gpu = s_m_gpu;
#pragma unroll
    for (int it = 0; it < IPT; ++it)
      if (m_gpu > 0 && it * RT + tid == (int)m_gpu - 1) s_gpu_part = S[it];
    __syncthreads();
    const uint64_t gpu_part = s_gpu_part;
    c = 0;
#pragma unroll
    for (int it = 0; it < IPT; ++it) {
      const uint32_t r = it * RT + tid;
      if (r >= m_gpu && r < P && S[it] - gpu_part <= a.cpu_bytes) ++c;
    }
    add_to(&s_m_cpu, c);
    __syncthreads();
    const uint32_t m_cpu = s_m_cpu, upper = m_gpu + m_cpu;
    uint32_t m_ssd = 0;
    if (ssd) {  // Sec. 7.1: the run after the CPU tier's, within the SSD budget
#pragma unroll
      for (int it = 0; it < IPT; ++it)
        if (upper > 0 && it * RT + tid == (int)upper - 1) s_upper_part = S[it];
      __syncthreads();
      const uint64_t upper_part = s_upper_part;
      c = 0;
#pragma unroll
      for (int it = 0; it < IPT; ++it) {
        const uint32_t r = it * RT + tid;
        if (r >= upper && r < P && S[it] - upper_part <= a.ssd_bytes) ++c;
      }
      add_to(&s_m_ssd, c);
      __syncthreads();
      m_ssd = s_m_ssd;
    }
#pragma unroll
    for (int it = 0; it < IPT; ++it) {
      const uint32_t r = it * RT + tid;
      s_tier[r] = r < m_gpu ? MORI_TIER_GPU
                : r < upper ? MORI_TIER_CPU
                : r < upper + m_ssd ? MORI_TIER_SSD : MORI_TIER_WAIT;
    }
  } else {
    // Greedy in rank order: the first tier that still has room.  Whether a
    // program fits a tier depends on that tier's room alone, so 64 ranks at a
    // time are offered to each tier in turn.
    __syncthreads();
    if (wid == 0) {
      uint64_t room_gpu = a.gpu_bytes / a.block_bytes, room_cpu = a.cpu_bytes / a.block_bytes;
      uint64_t room_ssd = a.ssd_bytes / a.block_bytes;
      uint32_t ng = 0, nc = 0, ns = 0;
      for (uint32_t c = 0; c < P; c += 64) {
        const bool valid = c + lane < P;
        const uint64_t b = valid ? s_id[c + lane] : 0u;
        const uint64_t all = __ballot(valid);
        const uint64_t gpu = take_fitting(all, b, room_gpu);
        const uint64_t cpu = take_fitting(all & ~gpu, b, room_cpu);
        const uint64_t sd = ssd ? take_fitting(all & ~(gpu | cpu), b, room_ssd) : 0ull;
        if (valid)
          s_tier[c + lane] = (gpu >> lane) & 1u ? MORI_TIER_GPU
                           : (cpu >> lane) & 1u ? MORI_TIER_CPU
                           : (sd >> lane) & 1u ? MORI_TIER_SSD : MORI_TIER_WAIT;
        ng += (uint32_t)__popcll(gpu);
        nc += (uint32_t)__popcll(cpu);
        ns += (uint32_t)__popcll(sd);
      }
      if (lane == 0) {
        s_m_gpu = ng;
        s_m_cpu = nc;
        s_m_ssd = ns;
      }
    }
  }
  __syncthreads();

  // ---- 4. sticky diff: categories, lists in rank order, bases -----------
  // scans: pages_out, pages_in, pages_admit, n_out | n_in << 16, n_admit_gpu
  // Global stores wait until after the last barrier: a barrier waits for the
  // stores still in flight, so stores issued earlier would stall every one.
  uint32_t v[IPT][5], ex[IPT][5], tot[5];
  uint8_t catv[IPT], tnewv[IPT];
  uint32_t n_drop = 0, n_ac = 0;  // dropped: from the GPU | from the CPU << 16
  uint32_t gpu_after = 0, cpu_after = 0, ssd_after = 0;  // blocks
#pragma unroll
  for (int it = 0; it < IPT; ++it) {
    const uint32_t r = it * RT + tid;
#pragma unroll
    for (int n = 0; n < 5; ++n) v[it][n] = 0;
    catv[it] = MORI_CAT_KEPT;
    if (r < P) {
      const uint32_t p = id[it];
      const uint8_t told = s_told[p], tnew = s_tier[r];
      const uint8_t c = category(told, tnew);
      catv[it] = c;
      tnewv[it] = tnew;
      if (c == MORI_CAT_OUT) v[it][0] = nb[it], v[it][3] = 1u;
      if (c == MORI_CAT_IN) v[it][1] = nb[it], v[it][3] = 1u << 16;
      if (c == MORI_CAT_ADMIT_GPU) v[it][2] = nb[it], v[it][4] = 1u;
      if (c == MORI_CAT_DROP_GPU) n_drop += 1u;
      if (c == MORI_CAT_DROP_CPU) n_drop += 1u << 16;
      if (c == MORI_CAT_ADMIT_CPU) ++n_ac;
      if (tnew == MORI_TIER_GPU) gpu_after += nb[it];
      if (tnew == MORI_TIER_CPU) cpu_after += nb[it];
      if (tnew == MORI_TIER_SSD) ssd_after += nb[it];
    }
  }
  scan_slices<NW, IPT, 5>(v, ex, s_tot, tot);
  const uint32_t pages_out = tot[0], pages_in = tot[1], pages_admit = tot[2];
  const uint32_t n_out = tot[3] & 0xFFFFu, n_in = tot[3] >> 16, n_admit = tot[4];
  // program-indexed staging, so the per-program stores below are coalesced:
  // the new tier and the page base by program id (every read of the
  // rank-indexed s_tier and s_nblk came before the scan's first barrier)
#pragma unroll
  for (int it = 0; it < IPT; ++it) {
    const uint32_t r = it * RT + tid;
    if (r >= P) continue;
    const uint32_t p = id[it];
    s_tier[p] = tnewv[it];
    if (catv[it] == MORI_CAT_OUT) s_nblk[p] = ex[it][0];
    if (catv[it] == MORI_CAT_IN) s_nblk[p] = ex[it][1];
    if (catv[it] == MORI_CAT_ADMIT_GPU) s_nblk[p] = pages_in + ex[it][2];
  }
  add_to(&s_n_drop, n_drop);
  add_to(&s_n_admit_cpu, n_ac);
  add_to(&s_gpu_after, gpu_after);
  add_to(&s_cpu_after, cpu_after);
  if (ssd) add_to(&s_ssd_after, ssd_after);
  __syncthreads();

  // ---- 5. the plan's stores ------------------------------------------------
  // by rank: order, prefix and the swap lists
#pragma unroll
  for (int it = 0; it < IPT; ++it) {
    const uint32_t r = it * RT + tid;
    if (r >= P) continue;
    const uint32_t p = id[it];
    a.order[r] = p;
    a.prefix[r] = S[it];
    *host_mirror(a, a.order + r) = p;
    *host_mirror(a, a.prefix + r) = S[it];
    const uint32_t idx_out = ex[it][3] & 0xFFFFu, idx_in = ex[it][3] >> 16;
    if (catv[it] == MORI_CAT_OUT) {
      const uint32_t pg = ex[it][0];
      a.ord[p] = idx_out;
      a.out_prog[idx_out] = p;
      a.out_pg_base[idx_out] = pg;
      *host_mirror(a, a.out_prog + idx_out) = p;
      *host_mirror(a, a.out_pg_base + idx_out) = pg;
    }
    if (catv[it] == MORI_CAT_IN) {  // programs promoted from the CPU (or SSD) tier take the first slots (Sec. 4.3.1)
      const uint32_t pg = ex[it][1];
      a.ord[p] = idx_in;
      a.in_prog[idx_in] = p;
      a.in_pg_base[idx_in] = pg;
      a.slot_base[idx_in] = pg;
      a.slot_prog[idx_in] = p;
      *host_mirror(a, a.in_prog + idx_in) = p;
      *host_mirror(a, a.in_pg_base + idx_in) = pg;
    }
    if (catv[it] == MORI_CAT_ADMIT_GPU) {  // then the programs admitted from Waiting: priority (2)
      const uint32_t idx = n_in + ex[it][4];
      a.slot_base[idx] = pages_in + ex[it][2];
      a.slot_prog[idx] = p;
    }
  }
  // by program id: tiers, categories and the page bases (swap-outs from their
  // first released page, swap-ins from theirs, then the programs admitted from
  // Waiting after every swap-in: priority (2))
#pragma unroll
  for (int it = 0; it < IPT; ++it) {
    const uint32_t x = it * RT + tid;
    if (x >= P) continue;
    const uint8_t told = s_told[x], tnew = s_tier[x], c = category(told, tnew);
    a.tier_old[x] = told;
    a.tier_new[x] = tnew;
    a.cat[x] = c;
    *host_mirror(a, a.tier_old + x) = told;
    *host_mirror(a, a.tier_new + x) = tnew;
    *host_mirror(a, a.cat + x) = c;
    if (c == MORI_CAT_OUT || c == MORI_CAT_IN || c == MORI_CAT_ADMIT_GPU) a.base[x] = s_nblk[x];
  }
  if (tid == 0) {
    a.out_pg_base[n_out] = pages_out;
    a.in_pg_base[n_in] = pages_in;
    *host_mirror(a, a.out_pg_base + n_out) = pages_out;
    *host_mirror(a, a.in_pg_base + n_in) = pages_in;
    DevSummary z = {};  // the page fields follow in the page kernels, which mirror the summary
    z.num_programs = P;
    z.m_gpu = s_m_gpu;
    z.m_cpu = s_m_cpu;
    z.m_ssd = s_m_ssd;
    z.n_out = n_out;
    z.n_in = n_in;
    z.n_drop_gpu = s_n_drop & 0xFFFFu;
    z.n_drop_cpu = s_n_drop >> 16;
    z.n_admit_gpu = n_admit;
    z.n_admit_cpu = s_n_admit_cpu;
    z.pages_out = pages_out;
    z.pages_in = pages_in;
    z.pages_admit = pages_admit;
    z.bytes_out = (uint64_t)pages_out * a.block_bytes;
    z.bytes_in = (uint64_t)pages_in * a.block_bytes;
    z.gpu_bytes_after = (uint64_t)s_gpu_after * a.block_bytes;
    z.cpu_bytes_after = (uint64_t)s_cpu_after * a.block_bytes;
    z.ssd_bytes_after = (uint64_t)s_ssd_after * a.block_bytes;
    z.need = (uint64_t)pages_in + pages_admit;
    *a.sum = z;
    a.swap_err[0] = a.swap_err[1] = 0;
  }
}

}  // namespace

hipError_t launch_rank(const PlanArgs& a, hipStream_t s) {
  static_assert(1024 * 4 == (int)MORI_MAX_PROGRAMS, "the large shape holds every program");
  // workgroup 0 ranks; the others (about two table entries per thread, at most
  // 2^21 threads in all) find the pages' owners.  With at most 2048 workgroups
  // whatever their size, the one-wave shape kept too few accesses in flight: a
  // pair of plans of 64 programs over 1 M, 2 M, 4 M pages 119, 177, 275 us, with
  // the bound on threads 109, 147, 211; of 256 over 4 M 238 -> 215.
  auto grid = [&](uint32_t rt) {
    const uint64_t g = ((uint64_t)a.tbl_len + 2ull * rt - 1) / (2ull * rt), most = (1u << 21) / rt;
    return dim3(1 + (uint32_t)(g < most ? g : most));
  };
  const bool counted = a.P > SORT_MAX_PROGRAMS || (uint64_t)a.P * a.k > SORT_MAX_CYCLES;
  if (counted) {
    hipLaunchKernelGGL(program_keys_kernel, dim3((a.P + KEY_WG - 1) / KEY_WG), dim3(KEY_WG), 0, s, a);
    hipLaunchKernelGGL(program_rank_kernel, dim3((a.P + RANK_WG / 64 - 1) / (RANK_WG / 64)), dim3(RANK_WG), 0, s, a);
  }
  if (a.P > 1024) hipLaunchKernelGGL((rank_partition_kernel<1024, 4, true>), grid(1024), dim3(1024), 0, s, a);
  else if (counted) hipLaunchKernelGGL((rank_partition_kernel<1024, 1, true>), grid(1024), dim3(1024), 0, s, a);
  else if (a.P <= 64) hipLaunchKernelGGL((rank_partition_kernel<64, 1, false>), grid(64), dim3(64), 0, s, a);
  else if (a.P <= 256) hipLaunchKernelGGL((rank_partition_kernel<256, 1, false>), grid(256), dim3(256), 0, s, a);
  else hipLaunchKernelGGL((rank_partition_kernel<1024, 1, false>), grid(1024), dim3(1024), 0, s, a);
  return hipGetLastError();
}

}  // namespace mori
