// Multi-replica admission of the shared Waiting queue (host code, no GPU work).
//
// Each replica keeps its own GPU and CPU queues and one Waiting queue is shared
// by all of them (Sec. 4.1).  Programs promoted from a replica's CPU tier stay
// on that replica (cache affinity) and are handled by its own plan; Waiting
// programs have no KV anywhere and are bin-packed across the replicas' free
// GPU capacity (Sec. 4.3.1): candidates in decreasing size, each onto the
// replica with the most room that holds it, or with MORI_ADMIT_BEST_FIT onto
// the one with the least such room.
//
// Both halves were bound by mispredicted compares and by a tree node freed and
// allocated per admission: 4096 programs on 64 replicas took 142 us with an
// indirect comparison sort and an ordered set, 30 with radix passes and flat
// arrays.
#include <algorithm>
#include <cstring>
#include <utility>
#include <vector>

#include "mori.h"

namespace {

struct Candidate {
  uint64_t order;     // ~bytes: larger KV first
  uint32_t idleness;  // its bits: ordered like the values, which are not negative
  uint32_t id;
};

inline bool before(const Candidate& x, const Candidate& y) {
  if (x.order != y.order) return x.order < y.order;
  if (x.idleness != y.idleness) return x.idleness < y.idleness;
  return x.id < y.id;
}

// Below this a comparison sort is faster than the radix passes and their 256
// counters (a call with lists of about 25 candidates 1.2 us against 2.2, of
// about 90 6.0 against 5.6, of about 180 9.6 against 7.2).
constexpr size_t RADIX_MIN = 96;

// Sorts by `before`; c comes in id order.  Stable byte-wise radix passes over
// the bits of the sizes that differ (they are multiples of a page, so 4 or 5
// passes), then the few runs of equal sizes by idleness.
void sort_candidates(std::vector<Candidate>& c) {
  if (c.size() < RADIX_MIN) {
    std::sort(c.begin(), c.end(), before);
    return;
  }
  uint64_t varying = 0;
  for (const Candidate& x : c) varying |= x.order ^ c[0].order;
  std::vector<Candidate> other(c.size());
  while (varying) {
    const int shift = __builtin_ctzll(varying);
    uint32_t at[256] = {};
    for (const Candidate& x : c) ++at[(x.order >> shift) & 255u];
    uint32_t sum = 0;
    for (uint32_t& n : at) sum += std::exchange(n, sum);
    for (const Candidate& x : c) other[at[(x.order >> shift) & 255u]++] = x;
    c.swap(other);
    varying &= ~(uint64_t{255} << shift);
  }
  for (size_t i = 0, j; i < c.size(); i = j) {
    for (j = i + 1; j < c.size() && c[j].order == c[i].order;) ++j;
    if (j - i > 1) std::sort(c.begin() + i, c.begin() + j, before);
  }
}

// The replica with the most room, the lowest one on ties: a tree of winners
// over the rooms, whose update compares once a level without a branch.
class MostRoom {
 public:
  MostRoom(const uint64_t* room, uint32_t R) {
    while (leaves_ < R) leaves_ *= 2;
    node_.assign(2 * leaves_, {0, 0});
    for (uint32_t r = 0; r < leaves_; ++r) node_[leaves_ + r] = {r < R ? room[r] : 0, r};
    for (uint32_t n = leaves_ - 1; n > 0; --n) node_[n] = winner(n);
  }
  std::pair<uint64_t, uint32_t> top() const { return node_[1]; }
  void set(uint32_t r, uint64_t room) {
    node_[leaves_ + r].first = room;
    for (uint32_t n = (leaves_ + r) / 2; n > 0; n /= 2) node_[n] = winner(n);
  }

 private:
  // the left child wins ties: it holds the lower replicas (and no padding, which comes last)
  std::pair<uint64_t, uint32_t> winner(uint32_t n) const {
    return node_[2 * n + (node_[2 * n + 1].first > node_[2 * n].first)];
  }
  uint32_t leaves_ = 1;
  std::vector<std::pair<uint64_t, uint32_t>> node_;
};

}  // namespace

extern "C" int mori_replica_admit(uint32_t num_programs, const uint64_t* bytes, const float* idleness,
                                  const uint8_t* status, uint32_t num_replicas, const uint64_t* room,
                                  uint32_t flags, int32_t* replica, uint64_t* room_after) {
  const uint32_t P = num_programs, R = num_replicas;
  if (R == 0 || R > MORI_MAX_REPLICAS || !room || !room_after) return MORI_EINVAL;
  if (P && (!bytes || !idleness || !status || !replica)) return MORI_EINVAL;
  if (flags & ~MORI_ADMIT_BEST_FIT) return MORI_EINVAL;
  for (uint32_t p = 0; p < P; ++p)
    if (status[p] > MORI_ST_NEW || !(idleness[p] >= 0.0f && idleness[p] <= 1.0f)) return MORI_EINVAL;

  // returning programs before new arrivals; larger KV first; lower idleness; lower id
  std::vector<Candidate> cand[2];
  for (auto& c : cand) c.reserve(P);
  for (uint32_t p = 0; p < P; ++p) {
    if (status[p] == MORI_ST_ACTING) continue;  // in a tool call, nothing to admit
    const float v = idleness[p] + 0.0f;         // a negative zero is +0
    Candidate c{~bytes[p], 0, p};
    std::memcpy(&c.idleness, &v, sizeof v);
    cand[status[p] == MORI_ST_NEW].push_back(c);
  }
  for (auto& c : cand) sort_candidates(c);

  std::memmove(room_after, room, sizeof(uint64_t) * R);
  for (uint32_t p = 0; p < P; ++p) replica[p] = -1;
  if (!(flags & MORI_ADMIT_BEST_FIT)) {
    MostRoom most(room_after, R);
    for (const auto& list : cand)
      for (const Candidate& c : list) {
        const uint64_t b = ~c.order;
        const auto [left, r] = most.top();
        if (left < b) continue;  // fits nowhere: stays waiting
        replica[c.id] = static_cast<int32_t>(r);
        most.set(r, room_after[r] = left - b);
      }
    return MORI_OK;
  }
  std::vector<std::pair<uint64_t, uint32_t>> free_room(R);  // (room, replica), ascending
  for (uint32_t r = 0; r < R; ++r) free_room[r] = {room_after[r], r};
  std::sort(free_room.begin(), free_room.end());
  for (const auto& list : cand)
    for (const Candidate& c : list) {
      const uint64_t b = ~c.order;
      // least room that holds it, lowest replica on ties
      const auto it = std::lower_bound(free_room.begin(), free_room.end(), std::make_pair(b, 0u));
      if (it == free_room.end()) continue;
      const uint32_t r = it->second;
      const std::pair<uint64_t, uint32_t> now(room_after[r] = it->first - b, r);
      const auto to = std::lower_bound(free_room.begin(), it, now);
      std::move_backward(to, it, it + 1);
      *to = now;
      replica[c.id] = static_cast<int32_t>(r);
    }
  return MORI_OK;
}
