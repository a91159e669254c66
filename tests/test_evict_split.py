"""The sample that splits the eviction order's blocks into buckets, on the
layouts that engines number blocks by: no bucket may outgrow the LDS sort."""
import numpy as np
import pytest

from evict_split import largest_bucket, lib, sample_blocks

SIZES = [8193, 16384, 32769, 70000, 131072, 300000, 700001, (1 << 20) - 361, 1 << 20]


def round_robin(N, rank_of_program):
    """Blocks dealt to programs in turn; a program's blocks follow one another
    in the order, programs in rank_of_program's."""
    P = rank_of_program.size
    count = np.full(P, N // P)
    count[:N % P] += 1
    by_rank = np.argsort(rank_of_program)
    first = np.empty(P, np.int64)
    first[by_rank] = np.cumsum(count[by_rank]) - count[by_rank]
    return lambda ids: first[ids % P] + ids // P


@pytest.mark.parametrize("N", SIZES)
def test_one_sample_in_each_stretch_of_ids(N):
    ids = sample_blocks(N)
    j = np.arange(ids.size, dtype=np.int64)
    assert (ids >= j * N // ids.size).all() and (ids < (j + 1) * N // ids.size).all()


@pytest.mark.parametrize("N", SIZES)
def test_round_robin_layouts(N):
    rng = np.random.default_rng(N)
    worst = 0
    for P in [*range(2, 130), *range(130, 8000, 13), 1005]:
        for rank in (np.arange(P), rng.permutation(P)):
            worst = max(worst, largest_bucket(N, round_robin(N, rank)))
    assert worst <= lib().bucket_cap(), worst


@pytest.mark.parametrize("bits", [15, 18, 20])
def test_strided_layouts(bits):
    """Time = block id x odd stride modulo a power of two."""
    N = 1 << bits
    worst = max(largest_bucket(N, lambda ids: ids * stride & (N - 1)) for stride in range(1, 30000, 6))
    assert worst <= lib().bucket_cap(), worst


@pytest.mark.parametrize("N", SIZES)
def test_contiguous_runs(N):
    """A program's blocks in one run of ids, programs in random order."""
    rng = np.random.default_rng(N)
    worst = 0
    for P in (2, 7, 64, 1000, 8000):
        edges = np.sort(rng.integers(0, N, size=P - 1))
        start, length = np.concatenate([[0], edges]), np.diff(np.concatenate([[0], edges, [N]]))
        by_rank = rng.permutation(P)
        first = np.empty(P, np.int64)
        first[by_rank] = np.cumsum(length[by_rank]) - length[by_rank]

        def place(ids):
            p = np.searchsorted(edges, ids, side="right")
            return first[p] + ids - start[p]

        worst = max(worst, largest_bucket(N, place))
    assert worst <= lib().bucket_cap(), worst


def test_workspace_holds_every_form():
    """What the caller is asked for covers the form each size takes, and the
    bucket form's need never falls with more blocks (a fixed array sized for the
    most blocks holds any fewer)."""
    L = lib()
    sizes = [L.direct_max() + 1, 8500, 16384, 32768, 32769, 69938, 1 << 18, (1 << 18) + 1, 1 << 19, L.bucket_max()]
    need = [L.bucket_bytes(N) for N in sizes]
    assert need == sorted(need)
    assert all(L.workspace_bytes(N) >= n for N, n in zip(sizes, need))
    for N in (L.bucket_max() + 1, (1 << 21) + 5000, (1 << 32) - 1):
        assert L.workspace_bytes(N) >= L.radix_bytes(N) >= 32 * N
