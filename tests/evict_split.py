"""The eviction order's own arithmetic (csrc/evict_split.h) for tests: limits of
its forms, buckets, and the blocks it samples, compiled from the header."""
import ctypes
import functools
import os
import subprocess
import tempfile

import numpy as np

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2606_00866_amd", "csrc")

SOURCE = """
#include "evict_split.h"
using namespace mori;
extern "C" uint32_t direct_max() { return DIRECT_MAX; }
extern "C" uint32_t bucket_max() { return BUCKET_MAX; }
extern "C" uint32_t bucket_cap() { return BUCKET_CAP; }
extern "C" uint32_t buckets(uint32_t N) { return bucket_count(N); }
extern "C" uint32_t samples(uint32_t N) { return sample_count(bucket_count(N)); }
extern "C" uint64_t bucket_bytes(uint32_t N) { return bucket_layout(N).bytes; }
extern "C" uint64_t radix_bytes(uint32_t N) { return radix_layout(N).bytes; }
extern "C" uint64_t workspace_bytes(uint32_t N) { return evict_workspace_bytes(N); }
extern "C" void sampled(uint32_t N, int64_t* ids) {
  for (uint32_t j = 0, S = samples(N); j < S; ++j) ids[j] = sample_block(j, S, N);
}
"""


@functools.lru_cache(None)
def lib():
    with tempfile.TemporaryDirectory() as tmp:
        src, so = os.path.join(tmp, "split.cpp"), os.path.join(tmp, "split.so")
        with open(src, "w") as f:
            f.write(SOURCE)
        subprocess.run(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-I", CSRC, src, "-o", so], check=True)
        L = ctypes.CDLL(so)
    for f in (L.bucket_bytes, L.radix_bytes, L.workspace_bytes):
        f.argtypes, f.restype = [ctypes.c_uint32], ctypes.c_uint64
    return L


@functools.lru_cache(None)
def sample_blocks(N):
    """Block ids the bucket form samples, in id order."""
    ids = np.empty(lib().samples(N), np.int64)
    lib().sampled(N, ids.ctypes.data_as(ctypes.c_void_p))
    return ids


def bucket_starts(N, place):
    """Where each bucket begins in the order by (key, id), and N; place(ids):
    each block's place in that order."""
    B, at = lib().buckets(N), np.sort(place(sample_blocks(N)))
    return np.concatenate([[0], at[:: at.size // B][1:], [N]])


def largest_bucket(N, place):
    """Blocks in the largest bucket."""
    return int(np.diff(bucket_starts(N, place)).max())
