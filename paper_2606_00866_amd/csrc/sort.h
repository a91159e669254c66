// Sorting in one workgroup: waves sort 64 entries each in registers, then sorted
// lists in LDS are merged two by two.  An entry is a (key, id) pair, or PACKED
// one word that holds both (the id in the low bits): one compare and two
// registers instead of three and three.  Entries are distinct.
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
// end early or lie past m altogether; both its ends are clamped, because the
// compiler dropped the test of `sib < m ? min(L, m - sib) : 0` (it took the
// subtraction not to wrap) and the search read past the entries.
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

}  // namespace mori
