// Sorting in one workgroup: waves sort 64 entries each in registers, then sorted
// lists in LDS are merged two by two.  An entry is a (key, id) pair, or PACKED
// one word that holds both (the id in the low bits): one compare and two
// registers instead of three and three.  Entries are distinct.  Or an element's
// place is counted, by a wave that compares it with every key.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "wave.h"

namespace mori {

__device__ inline bool pair_less(uint64_t ka, uint32_t ia, uint64_t kb, uint32_t ib) {
  return ka < kb || (ka == kb && ia < ib);
}

template <bool PACKED>
__device__ inline bool entry_less(uint64_t ka, uint32_t ia, uint64_t kb, uint32_t ib) {
  return PACKED ? ka < kb : pair_less(ka, ia, kb, ib);
}

// A wave's 64 entries ascending by lane: a bitonic network.  n: entries that are
// not padding above every other one, in the lowest lanes; a network of the next
// power of two is enough for them.
template <bool PACKED>
__device__ inline void sort_wave(uint64_t& key, uint32_t& id, uint32_t n = 64) {
  const uint32_t lane = threadIdx.x & 63;
  auto step = [&](auto D, uint32_t size) {
    constexpr uint32_t d = decltype(D)::value;
    const uint64_t k = wave::swap_lanes<d>(key);
    const uint32_t i = PACKED ? 0u : wave::swap_lanes<d>(id);
    const bool low = (lane & d) == 0, up = (lane & size) == 0;
    if (entry_less<PACKED>(k, i, key, id) == (low == up)) {
      key = k;
      if (!PACKED) id = i;
    }
  };
#pragma unroll
  for (uint32_t size = 2; size <= 64; size <<= 1) {
    if (size / 2 >= n) break;  // uniform
    if (size >= 64) step(std::integral_constant<uint32_t, 32>(), size);
    if (size >= 32) step(std::integral_constant<uint32_t, 16>(), size);
    if (size >= 16) step(std::integral_constant<uint32_t, 8>(), size);
    if (size >= 8) step(std::integral_constant<uint32_t, 4>(), size);
    if (size >= 4) step(std::integral_constant<uint32_t, 2>(), size);
    step(std::integral_constant<uint32_t, 1>(), size);
  }
}

// Place of entry (key, id), now at x of s_key[0, m) (and s_id unless PACKED),
// when each list of L entries is merged with its sibling: its place in its own
// list plus, by binary search, the sibling's entries below it.  The sibling may
// end early or lie past m altogether, so both its ends are clamped.
template <bool PACKED>
__device__ inline uint32_t merged_place(const uint64_t* s_key, const uint32_t* s_id, uint32_t m, uint32_t L, uint32_t x,
                                        uint64_t key, uint32_t id) {
  const uint32_t own = x & ~(L - 1), sib = own ^ L, first = min(sib, m);
  uint32_t lo = first, hi = min(sib + L, m);
  while (lo < hi) {
    const uint32_t mid = (lo + hi) >> 1;
    const uint64_t k = s_key[mid];
    if (PACKED ? k < key : k < key || (k == key && s_id[mid] < id)) lo = mid + 1;
    else hi = mid;
  }
  return min(own, sib) + (x - own) + (lo - first);
}

// For E consecutive staged elements i0 .. i0 + E - 1 of one wave (i0 a multiple
// of E): how many staged keys come before each (lower key, or equal key and
// lower index) and with BYTES the sum of their sizes.  The keys come in chunks
// of 64, a multiple of GROUP of them; keys past the last element are all ones.
// The elements' keys are uniform, so a chunk costs a 64-bit compare against a
// scalar and an add of the carry per element.  Equal keys come first in lower
// groups of chunks, where the compare is with key + 1, not in higher ones,
// where it is with the key, and by index in the elements' own group.
constexpr uint32_t GROUP = 4;  // chunks whose loads are in flight together
template <int E, bool BYTES>
__device__ inline void count_before(const uint64_t* s_key, const uint32_t* s_size, uint32_t chunks, uint32_t i0,
                                    uint32_t (&rank)[E], uint64_t (&bytes)[E]) {
  const uint32_t lane = threadIdx.x & 63;
  uint64_t k[E], sum[E];
  uint32_t cnt[E];
#pragma unroll
  for (int e = 0; e < E; ++e) {
    k[e] = wave::uniform(s_key[i0 + e]);
    cnt[e] = 0;
    sum[e] = 0;
  }
  auto group = [&](uint32_t c0, auto limit) {
    uint64_t kj[GROUP];
    uint32_t sz[GROUP];
#pragma unroll
    for (uint32_t g = 0; g < GROUP; ++g) {
      kj[g] = s_key[(c0 + g) * 64 + lane];
      sz[g] = BYTES ? s_size[(c0 + g) * 64 + lane] : 0u;
    }
#pragma unroll
    for (uint32_t g = 0; g < GROUP; ++g)
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const bool before = kj[g] < limit(e, (c0 + g) * 64 + lane);
        cnt[e] += before;
        if (BYTES) sum[e] += before ? sz[g] : 0u;
      }
  };
  const uint32_t own = (uint32_t)__builtin_amdgcn_readfirstlane((int)(i0 / (64 * GROUP) * GROUP));
  for (uint32_t c = 0; c < own; c += GROUP) group(c, [&](int e, uint32_t) { return k[e] + 1; });
  group(own, [&](int e, uint32_t j) { return k[e] + (j < i0 + e); });
  for (uint32_t c = own + GROUP; c < chunks; c += GROUP) group(c, [&](int e, uint32_t) { return k[e]; });
#pragma unroll
  for (int e = 0; e < E; ++e) {
    rank[e] = wave::sum(cnt[e]);
    bytes[e] = BYTES ? wave::sum(sum[e]) : rank[e];
  }
}

}  // namespace mori
