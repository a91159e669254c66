"""libmori's multi-replica admission (host code behind the C ABI) against the
oracle, element by element, on random Waiting queues: up to 4096 programs
with ties in size and idleness, 1 to 1024 replicas, both replica rules; and its
argument checks.  No GPU is involved."""
import numpy as np
import pytest

from paper_2606_00866_amd import mori as M


@pytest.mark.parametrize("seed", range(40))
def test_matches_oracle(orc, seed):
    rng = np.random.default_rng(7000 + seed)
    P = int(rng.choice([0, 1, 7, 100, 1000, 4096]))
    R = int(rng.choice([1, 2, 3, 8, 64, 1024]))  # 1024: the maximum
    sizes = rng.integers(0, 40, P) * int(rng.choice([1, 2 << 20]))  # ties in size
    iota = rng.choice(np.array([0, 0.25, 0.5, 1], np.float32), P) if seed % 2 else rng.random(P).astype(np.float32)
    st = rng.choice(3, P, p=[0.5, 0.2, 0.3]).astype(np.uint8)
    room = (rng.integers(0, max(1, int(sizes.sum()) // max(R, 1) + 2), R)).astype(np.uint64)
    for flags in (0, M.MORI_ADMIT_BEST_FIT):
        rc, rep, after = M.mori_replica_admit(sizes, iota, st, room, flags)
        orc_rc, orc_rep, orc_after = orc.replica_admit(sizes, iota, st, room, orc.ADMIT_BEST_FIT if flags else 0)
        assert rc == M.MORI_OK and orc_rc == orc.OK
        assert np.array_equal(rep, orc_rep), (seed, flags)
        assert np.array_equal(after, orc_after)


@pytest.mark.parametrize("P", [200, 321, 5000])
@pytest.mark.parametrize("high", [40, 1 << 20, 1 << 40, 1 << 64])
def test_sizes_of_any_width(orc, P, high):
    """Sizes that differ in one to eight bytes (the radix passes), zeros of both
    signs among the idleness, and replica counts that are no power of two."""
    rng = np.random.default_rng([P, high % 1000003])
    sizes = rng.integers(0, high, P, dtype=np.uint64)
    iota = rng.choice(np.array([0.0, -0.0, 1e-40, 0.5], np.float32), P)
    st = rng.choice(3, P, p=[0.5, 0.2, 0.3]).astype(np.uint8)
    for R in (5, 77, 1023):
        room = rng.integers(0, high, R, dtype=np.uint64)
        for flags in (0, M.MORI_ADMIT_BEST_FIT):
            rc, rep, after = M.mori_replica_admit(sizes, iota, st, room, flags)
            orc_rc, orc_rep, orc_after = orc.replica_admit(sizes, iota, st, room, orc.ADMIT_BEST_FIT if flags else 0)
            assert rc == M.MORI_OK and orc_rc == orc.OK
            assert np.array_equal(rep, orc_rep) and np.array_equal(after, orc_after)


def test_argument_checks():
    one = dict(bytes_=[1], idleness=[0.5], status=[0], room=[4])

    def run(flags=0, **kw):
        d = dict(one, **kw)
        return M.mori_replica_admit(d["bytes_"], d["idleness"], d["status"], d["room"], flags)[0]

    assert run() == M.MORI_OK
    assert run(room=[]) == M.MORI_EINVAL
    assert run(room=np.zeros(M.MORI_MAX_REPLICAS + 1, np.uint64)) == M.MORI_EINVAL
    assert run(flags=2) == M.MORI_EINVAL
    assert run(status=[3]) == M.MORI_EINVAL
    assert run(idleness=[1.5]) == M.MORI_EINVAL
    assert run(idleness=[np.nan]) == M.MORI_EINVAL
    # no programs: room unchanged
    rc, rep, after = M.mori_replica_admit([], [], [], [5, 6])
    assert rc == M.MORI_OK and rep.size == 0 and after.tolist() == [5, 6]


def test_bench_inputs(orc):
    """The multi-replica leg of bench.py times these exact inputs."""
    import bench

    for P, R in bench.REPLICA_CASES:
        sizes, iota, status, room = bench.replica_inputs(np, P, R)
        for flags in (0, M.MORI_ADMIT_BEST_FIT):
            rc, rep, after = M.mori_replica_admit(sizes, iota, status, room, flags)
            orc_rc, orc_rep, orc_after = orc.replica_admit(sizes, iota, status, room,
                                                           orc.ADMIT_BEST_FIT if flags else 0)
            assert rc == M.MORI_OK and orc_rc == orc.OK
            assert np.array_equal(rep, orc_rep) and np.array_equal(after, orc_after)
            assert 0 < (rep >= 0).sum() < P  # some admitted, some left waiting
