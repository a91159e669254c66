// Internal declarations of libmori shared by the kernel files and the C ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/mori.h"

namespace mori {

// What the step does with a page.
constexpr uint32_t PC_KEPT = 0u;   // owned by a program that stays on the GPU
constexpr uint32_t PC_FREE = 1u;   // marked free in the caller's free map before the step
constexpr uint32_t PC_REL = 2u;    // owned by a program leaving the GPU, free at once
constexpr uint32_t PC_LATER = 3u;  // ... free only after the swap-out stream has passed: the swap-out
                                   // reads it, or its dropped program may still be running

constexpr int PAGE_TILE = 512;     // pages per workgroup in the page-allocation kernels (2 per thread;
                                   // measured: 0.5-1 us faster per plan than 1024, 2048 slower)

// Plan summary as kept on the device (the head of the plan blob, mirrored on the host).
struct DevSummary {
  uint32_t num_programs, m_gpu, m_cpu, m_ssd;
  uint32_t n_out, n_in, n_drop_gpu, n_drop_cpu, n_admit_gpu, n_admit_cpu;
  uint32_t error;
  uint64_t pages_out, pages_in, pages_admit;
  uint64_t pages_free_before, pages_released, pages_recycled, pages_free_after;
  uint64_t bytes_out, bytes_in, gpu_bytes_after, cpu_bytes_after, ssd_bytes_after;
  uint64_t need;  // pages_in + pages_admit
  uint64_t pages_dropped;  // released pages nothing reads any more: slots below free-before + this need no wait
};

// A registered memory range usable by the swap kernels.
struct DevRange {
  uint64_t host_base;  // address as the caller names it
  uint64_t bytes;
  uint64_t dev_base;   // the same memory as the GPU addresses it
  uint64_t is_device;  // 1: HBM, 0: pinned host memory
};

// Everything the plan kernels read and write.
struct PlanArgs {
  // caller-owned
  const float* window;
  const float* idleness;
  const uint8_t* status;
  const uint32_t* tbl_off;
  uint32_t* tbl;
  uint8_t* tier;
  uint8_t* free_map;
  uint32_t tbl_len, P, k, flags, NB, ntiles;
  uint64_t block_bytes, gpu_bytes, cpu_bytes, ssd_bytes;
  // context scratch: plan blob (mirrored to the host)
  DevSummary* sum;
  uint32_t* order;
  uint64_t* prefix;
  uint8_t* tier_old;
  uint8_t* tier_new;
  uint8_t* cat;
  uint32_t* out_prog;
  uint32_t* in_prog;
  uint32_t* out_pg_base;  // [n_out + 1] first out-page index of each out program
  uint32_t* in_pg_base;   // [n_in + 1] first slot of each in program
  // context scratch: device only
  uint64_t* key;          // per program: its key
  uint32_t* key_err;      // per 64 programs: what is wrong with their data
  uint64_t* rank_rec;     // by rank: program and what the placement reads of it
  uint32_t* base;         // per program: out-page base (OUT) or slot base (IN, ADMIT_GPU)
  uint64_t* owner;        // [NB] program << 32 | (table entry + 1) of each owned page, 0 between plans
  uint8_t* pcode;         // [NB] PC_* of each page
  uint32_t* page_err;     // ownership errors, 0 between plans
  uint32_t* slot_base;    // [n_in + n_admit_gpu] first slot of each program entering the GPU, in slot order
  uint32_t* slot_prog;    // [n_in + n_admit_gpu] that program
  uint32_t* out_src;      // [pages_out] old page of each out page index
  uint32_t* in_dst;       // [need] page of each slot
  uint32_t* ord;          // per program: its index in the swap-out or swap-in list (OUT, IN)
  uint32_t* out_ord;      // [pages_out] swap-out list index of each out page index
  uint32_t* in_ord;       // [pages_in] swap-in list index of each slot
  uint64_t* tile_cnt;     // [2 ntiles]: packed (free-before, dropped << 32), then free-later counts
  uint64_t* tile_base;    // [2 ntiles] exclusive prefixes of both halves of tile_cnt
  uint32_t* swap_err;     // [2] swap-out, swap-in address errors; cleared by every plan
  // The pinned host mirror of the plan blob, as the device addresses it: the
  // kernels that finish a part of the plan store it there too, so no copy of
  // the blob follows the plan.  Mirror address = blob address + host_delta.
  int64_t host_delta;
};

template <typename T>
__device__ inline T* host_mirror(const PlanArgs& a, T* blob_ptr) {
  return reinterpret_cast<T*>(reinterpret_cast<char*>(blob_ptr) + a.host_delta);
}

// Unit ranges of a kernel-direct swap, written by its translation (all zero
// after a failed plan): [0, total) is the whole direction, [0, first_end) the
// first part of a swap-in and [second_begin, total) the second.
struct SwapRange {
  uint64_t total, first_end, second_begin;
  uint64_t nf;  // slots below it need no wait
};

// Everything a swap kernel reads.
struct SwapArgs {
  uint8_t* pool;
  uint64_t NB, run;
  uint32_t LC;              // layers * planes
  const SwapRange* range;   // kernel-direct mode: this direction's unit ranges
  const uint32_t* prog;     // out_prog or in_prog
  const uint32_t* pg_base;  // out_pg_base or in_pg_base
  const uint32_t* pages;    // out_src (by out-page index) or in_dst (by slot)
  const uint32_t* ord;      // out_ord or in_ord: list index of each out-page index / slot
  const uint64_t* addr;     // device address of each program's host buffer
  const uint32_t* swap_err; // [2] address errors found by the swap-out's and the swap-in's translation
  uint8_t* staging;         // non-null: chunk staging buffer (copy-engine mode)
  uint64_t u_begin, u_end;  // staging mode: unit range of the chunk
  uint32_t part;            // swap-in: 0 all slots, 1 slots < free-before, 2 slots >= free-before
  uint32_t host_link;       // 1: the other side is pinned host memory (kernel-direct mode over the host link)
};

struct TranslateArgs {
  const DevSummary* sum;
  const uint32_t* pg_base;  // out_pg_base or in_pg_base
  const uint32_t* ord;      // out_ord or in_ord
  SwapRange* range;         // this direction's
  uint32_t LC;
  const uint32_t* prog;     // out_prog or in_prog (count n_out / n_in)
  int dir_in;               // 0 out, 1 in
  const uint32_t* tbl_off;
  uint64_t block_bytes;
  const uint64_t* addr_in;  // [P] caller addresses, in pinned host memory
  uint64_t* addr_out;       // [P] translated device addresses
  const DevRange* ranges;
  uint32_t nranges;
  uint32_t* swap_err;       // [2]: this direction's word is swap_err[dir_in]
};

// launchers (return the launch error)
hipError_t launch_rank(const PlanArgs& a, hipStream_t s);
hipError_t launch_clear_owner(const PlanArgs& a, hipStream_t s);
hipError_t launch_pages(const PlanArgs& a, hipStream_t s);
hipError_t launch_translate(const TranslateArgs& a, hipStream_t s);
hipError_t launch_swap_out(const SwapArgs& a, uint32_t grid, hipStream_t s);
hipError_t launch_swap_in(const SwapArgs& a, uint32_t grid, hipStream_t s);
uint32_t swap_runs_per_workgroup(uint64_t run);  // per pass of a kernel-direct swap between HBM buffers
hipError_t launch_evict(uint32_t N, const uint8_t* type, const uint64_t* last_access, const uint32_t* size,
                        uint64_t unit_bytes, uint32_t tier, uint64_t need, void* workspace, uint32_t* order,
                        uint64_t* prefix, uint32_t* result, hipStream_t s);

}  // namespace mori
