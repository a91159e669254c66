"""The eviction order at the limits of its three forms (direct counting, sorted
buckets, radix passes) and where the bucket form can go wrong: keys too wide to
pack with an id, equal keys throughout, and a sample that misses the
distribution, which leaves one bucket larger than a workgroup sorts in LDS."""
import numpy as np
import pytest
import torch

from evict_split import largest_bucket, lib, sample_blocks
from gpu_helpers import log
from oracle import oracle
from paper_2606_00866_amd import mori as M
from test_gpu_evict import check, run_gpu
from workload import eviction_blocks

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [1, 63, 64, 65, 256, 257, 4096, 4097, 8191, 8192, 8193, 12345, 32769, 262144, 262145,
                               524289, 1 << 20, (1 << 20) + 1])
def test_limits_of_the_forms(N):
    rng = np.random.default_rng(N)
    for var_size, horizon in ((True, 1 << 40), (False, 1 << 61)):
        typ, la, size = eviction_blocks(rng, N, programs=min(N, 700), tie_frac=0.5, horizon=horizon, var_size=var_size)
        total = N if size is None else int(size.astype(np.int64).sum())
        log(f"evict N={N} sizes={var_size}")
        check(typ, la, size, 7, N % 2, (total // 2) * 7 + 1)


@pytest.mark.parametrize("N", [9000, 70000, 300000])
@pytest.mark.parametrize("kind", ["equal", "ascending", "descending", "spread", "zero sizes"])
def test_key_shapes_in_buckets(N, kind):
    """Equal keys, keys in and against id order, keys over the whole 62 bits
    with all types (buckets too wide to pack), and blocks of size zero."""
    rng = np.random.default_rng(N)
    typ, size = np.zeros(N, np.uint8), None
    la = np.full(N, 12345, np.uint64)
    if kind == "ascending":
        la = np.arange(N, dtype=np.uint64)
    elif kind == "descending":
        la = np.arange(N, dtype=np.uint64)[::-1].copy() << np.uint64(20)
    elif kind == "spread":
        typ = rng.integers(0, 3, size=N).astype(np.uint8)
        la = rng.integers(0, 1 << 62, size=N).astype(np.uint64)
    elif kind == "zero sizes":
        la = rng.integers(0, 50, size=N).astype(np.uint64)
        size = rng.integers(0, 2, size=N).astype(np.uint32)
    log(f"evict {kind} N={N}")
    check(typ, la, size, 16, 0, 16 * (N // 4))


@pytest.mark.parametrize("N", [300000, 1 << 20])
def test_regular_layouts(N):
    """Block ids dealt round-robin to 1005 programs, and strided times."""
    i = np.arange(N, dtype=np.uint64)
    log(f"evict layouts N={N}")
    check(np.ones(N, np.uint8), i % np.uint64(1005), None, 16, 0, 16 * (N // 3))
    check(np.ones(N, np.uint8), i * np.uint64(2391) & np.uint64(0xFFFFF), None, 16, 1, 16 * (N // 3))


@pytest.mark.parametrize("var_size", [False, True])
def test_bucket_larger_than_lds(var_size):
    """Every sampled block is old and all others share a few recent times, so
    the last bucket holds about 19 000 of 20 000 blocks."""
    N = 20000
    rng = np.random.default_rng(1)
    la = rng.integers(1 << 40, (1 << 40) + 100, size=N).astype(np.uint64)
    sampled = sample_blocks(N)
    la[sampled] = rng.integers(0, 1000, size=sampled.size).astype(np.uint64)
    place = np.empty(N, np.int64)
    place[np.argsort(la, kind="stable")] = np.arange(N)
    assert largest_bucket(N, lambda ids: place[ids]) > lib().bucket_cap()
    size = rng.integers(1, 9, size=N).astype(np.uint32) if var_size else None
    check(np.ones(N, np.uint8), la, size, 3, 1, 3 * (N // 2))


@pytest.mark.parametrize("kind", ["first", "middle", "two", "ties", "wide"])
@pytest.mark.parametrize("N", [15000, 33000, 300000, 1 << 20])
def test_buckets_cut_into_pieces(N, kind):
    """Blocks that no sample meets lie in one bucket (before all sampled blocks,
    amid them, or in two stretches between them), with times of their own, a few
    tied times (the pieces end between ids) or keys over all types and times."""
    rng = np.random.default_rng(N)
    sampled = sample_blocks(N)
    typ = np.ones(N, np.uint8)
    base = np.uint64(1 << 41)
    la = base + rng.integers(0, 8 if kind == "ties" else 1 << 40, size=N).astype(np.uint64)
    outer = rng.integers(0, 1 << 40, size=sampled.size).astype(np.uint64)
    above = np.arange(sampled.size) % 2 == 1
    if kind == "first":
        above[:] = True
    la[sampled] = outer + np.where(above, np.uint64(1 << 43), np.uint64(0))
    if kind == "two":
        la[np.arange(N) % 2 == 1] += np.uint64(1 << 42)
        third = np.arange(sampled.size) % 3
        la[sampled] = outer + np.array([0, (1 << 41) + (1 << 40), 1 << 43], np.uint64)[third]
    if kind == "wide":
        typ = rng.integers(0, 3, size=N).astype(np.uint8)
        la = rng.integers(1 << 20, 1 << 62, size=N).astype(np.uint64)
        typ[sampled] = np.where(above, 0, 2)
        la[sampled] = np.where(above, np.uint64((1 << 62) - 1), np.uint64(0))
    place = np.empty(N, np.int64)
    place[np.lexsort((la, 2 - typ.astype(np.int64)))] = np.arange(N)
    assert largest_bucket(N, lambda ids: place[ids]) > lib().bucket_cap()
    size = rng.integers(0, 9, size=N).astype(np.uint32)
    log(f"evict {kind} pieces N={N}")
    check(typ, la, size, 3, 0, 3 * (int(size.sum()) // 2))


@pytest.mark.parametrize("span", [(1 << 44) - 2, (1 << 44) - 1, 1 << 44])
def test_packing_limit(span):
    """The last of 2^20 blocks, all others of one time, is `span` newer: at
    2^44 - 1 its key and id in one word would equal the bucket's padding."""
    N = 1 << 20
    la = np.full(N, 99, np.uint64)
    la[N - 1] = 99 + span
    log(f"evict span={span}")
    check(np.zeros(N, np.uint8), la, None, 16, 0, 16 * (N - 1) + 1)


@pytest.mark.parametrize("N", [3000, 50000, (1 << 20) + 5000, (1 << 21) + 5000])
def test_invalid_block_and_no_prefix(N):
    rng = np.random.default_rng(N)
    typ, la, size = eviction_blocks(rng, N, programs=40, tie_frac=0.5, var_size=True)
    bad = typ.copy()
    bad[N - 1] = 200
    _, _, res = run_gpu(bad, la, size, 1, 0, 10)
    assert list(res) == [0, M.MORI_DEV_BAD_BLOCK]
    rc, o_order, _, o_count = oracle.evict_order(typ, la, 0, N, size=size, unit_bytes=1)
    t, l, s = (torch.from_numpy(a).cuda() for a in (typ, la.view(np.int64), size.view(np.int32)))
    wbytes = M.mori_evict_workspace(N)[1]
    ws = torch.empty(wbytes, dtype=torch.uint8, device="cuda")
    order = torch.empty(N, dtype=torch.int32, device="cuda")
    res = torch.zeros(2, dtype=torch.int32, device="cuda")
    blk = M.mori_blocks(N, t.data_ptr(), l.data_ptr(), s.data_ptr(), 1)
    assert M.mori_evict_order(blk, 0, N, ws.data_ptr(), wbytes, order.data_ptr(), 0, res.data_ptr(),
                              torch.cuda.current_stream().cuda_stream) == M.MORI_OK
    torch.cuda.synchronize()
    assert np.array_equal(order.cpu().numpy().view(np.uint32), o_order) and res.cpu().tolist() == [o_count, 0]
