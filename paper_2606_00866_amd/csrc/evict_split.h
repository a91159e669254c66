// How the eviction order chooses its form, lays out its workspace and splits
// blocks into buckets: plain arithmetic, for the kernels and for host code alike.
#pragma once
#include <stdint.h>

namespace mori {

// Direct counting grows with the square: 15.3 us at 8 192 blocks against 21 for
// the buckets, about 24 at 10 240, and the keys no longer fit LDS twice as far.
constexpr uint32_t DIRECT_MAX = 8192;
// The bucket form ends where a packed entry runs out of id bits.
constexpr uint32_t BUCKET_ID_BITS = 20;
constexpr uint32_t BUCKET_MAX = 1u << BUCKET_ID_BITS;
constexpr uint32_t BUCKETS_MAX = 1024;
// Eight samples a bucket, at least 1024 (more balance the buckets better, but
// ranking them grows with the square: 4096 for 256 buckets 1.5 us slower).
constexpr uint32_t SAMPLES_PER_BUCKET = 8, SAMPLES_MIN = 1024;
constexpr uint32_t SAMPLES_MAX = SAMPLES_PER_BUCKET * BUCKETS_MAX;
// Blocks per bucket aimed at while there are buckets left: 1024 is 9 us slower
// at 131 072 blocks and 5 us at 2^19, 256 within 3 us either way.
constexpr uint32_t BUCKET_AVG = 512;
constexpr uint32_t BUCKET_CAP = 6144;  // a bucket of up to this many blocks is sorted in LDS

// Buckets for N blocks (a power of two) and samples for them (a multiple).
constexpr uint32_t bucket_count(uint32_t N) {
  uint32_t B = 64;
  while (B < BUCKETS_MAX && (uint64_t)B * BUCKET_AVG < N) B *= 2;
  return B;
}
constexpr uint32_t sample_count(uint32_t B) {
  return B * SAMPLES_PER_BUCKET > SAMPLES_MIN ? B * SAMPLES_PER_BUCKET : SAMPLES_MIN;
}

// Every bit of x reaches the high bits: multiplications carry upwards, the
// shifts bring the result down for the next one.
constexpr uint32_t mix(uint32_t x) {
  constexpr uint32_t ODD = 0x9E3779B1u;  // near 2^32 / golden ratio
  x = (x + 1u) * ODD;
  x = (x ^ (x >> 16)) * ODD;
  return (x ^ (x >> 15)) * ODD;
}

// Sample j's block: a pseudo-random one of the j-th of S equal stretches of
// block ids (so sample order is id order).  Engines number blocks regularly
// (round-robin over programs, strided), and a choice whose steps from stretch
// to stretch are regular too resonates with that: with the high bits of one
// multiplication, strided times left buckets of up to 689 881 of 2^20 blocks and
// round-robin ids of up to 340 516; with this mix none is above 4 400.
constexpr uint32_t sample_block(uint32_t j, uint32_t S, uint32_t N) {
  const uint32_t lo = (uint32_t)((uint64_t)j * N / S), hi = (uint32_t)((uint64_t)(j + 1) * N / S);
  return lo + (uint32_t)(((uint64_t)mix(j) * (hi - lo)) >> 32);
}

// A form's pieces of the workspace, as byte offsets in it; `bytes` is where the
// last one ends.  Pieces are 256-B aligned.
class Pieces {
 public:
  constexpr uint64_t take(uint64_t bytes) {
    const uint64_t at = end_;
    end_ += (bytes + 255) & ~255ull;
    return at;
  }
  constexpr uint64_t end() const { return end_; }

 private:
  uint64_t end_ = 0;
};

struct BucketLayout {
  uint64_t key, id, spl_key, units, spl_id, count, taken, first, below, over, sample, err, bytes;
};
constexpr BucketLayout bucket_layout(uint32_t N) {
  Pieces p;
  BucketLayout l{};
  l.key = p.take(8ull * N);
  l.id = p.take(4ull * N);
  l.spl_key = p.take(8 * BUCKETS_MAX);
  l.units = p.take(8 * BUCKETS_MAX);
  l.spl_id = p.take(4 * BUCKETS_MAX);
  l.count = p.take(4 * BUCKETS_MAX);
  l.taken = p.take(4 * BUCKETS_MAX);
  l.first = p.take(4 * (BUCKETS_MAX + 1));
  l.below = p.take(8 * (BUCKETS_MAX + 1));
  l.over = p.take(4);
  l.sample = p.take(8 * SAMPLES_MAX);
  l.err = p.take(8);
  l.bytes = p.end();
  return l;
}

// Radix tiles: workgroup size and keys per thread.
constexpr int EVICT_WG = 256;
constexpr int EVICT_KEYS_PER_THREAD = 8;
constexpr uint32_t radix_tiles(uint32_t N) {
  constexpr uint64_t tile = (uint64_t)EVICT_WG * EVICT_KEYS_PER_THREAD;
  return (uint32_t)(((uint64_t)N + tile - 1) / tile);
}
struct RadixLayout {
  uint64_t keys[2], vals[2], hist, dtot, tile_sum, prefix, misc, bytes;
};
constexpr RadixLayout radix_layout(uint32_t N) {
  const uint32_t ntiles = radix_tiles(N);
  Pieces p;
  RadixLayout l{};
  l.keys[0] = p.take(8ull * N);
  l.keys[1] = p.take(8ull * N);
  l.vals[0] = p.take(4ull * N);
  l.vals[1] = p.take(4ull * N);
  l.hist = p.take(4ull * 256 * ntiles);
  l.dtot = p.take(4 * 256);
  l.tile_sum = p.take(8ull * ntiles);
  l.prefix = p.take(8ull * N);
  l.misc = p.take(8 * 4);
  l.bytes = p.end();
  return l;
}

// What mori_evict_order asks of its caller: one formula for all N, above every
// form's need (direct counting uses no workspace, the buckets 12 B a block and
// under 150 KB, the radix passes about 32.5 B a block).
constexpr uint64_t evict_workspace_bytes(uint32_t N) { return radix_layout(N).bytes + (1u << 20); }

}  // namespace mori
