"""The rank order for program counts whose sorted lists of 64, 128, 256 or 512
have no sibling to merge with, run after a plan of 1024 programs has filled the
workgroup's memory, with keys that pack with the id into one word and, through
one new arrival of 2^19 blocks, keys that do not; and above 1024 programs, where
several workgroups key and rank them, at the remainders of 16, 64, 256 and 1024
programs, with programs that are rejected in any of the workgroups."""
import numpy as np
import pytest
import torch

from gpu_helpers import log
from paper_2606_00866_amd import mori as M

pytestmark = pytest.mark.gpu


def rank_order(ctx, keep, idleness, tier, status, nblk, incremental):
    P = idleness.size
    off = np.zeros(P + 1, np.uint32)
    off[1:] = np.cumsum(nblk)
    dev = [torch.from_numpy(a).cuda() for a in (idleness, tier, status, off.view(np.int32),
                                                np.full(max(int(off[-1]), 1), -1, np.int32))]
    free = torch.ones(64, dtype=torch.uint8, device="cuda")
    keep += dev + [free]
    flags = M.MORI_F_IDLENESS_GIVEN | (M.MORI_F_INCREMENTAL if incremental else 0)
    prog = M.mori_programs(P, 0, None, dev[0].data_ptr(), dev[2].data_ptr(), dev[3].data_ptr(), int(off[-1]),
                           dev[4].data_ptr(), dev[1].data_ptr(), free.data_ptr())
    torch.cuda.synchronize()
    assert M.mori_rank_partition(ctx, prog, M.mori_budget(0, 0, flags, 0)) == M.MORI_OK
    rc, plan = M.mori_plan_wait(ctx)
    if rc != M.MORI_OK:
        assert rc == M.MORI_EDEVICE
        return plan.device_error
    return np.ctypeslib.as_array(plan.order, shape=(P,)).copy()


@pytest.mark.parametrize("P", [2, 63, 64, 65, 129, 200, 256, 257, 321, 450, 577, 700, 833, 1000, 1024,
                               1025, 1041, 1500, 2048, 2305, 4033, 4095, 4096])
@pytest.mark.parametrize("kind", ["boundary", "incremental", "wide"])
def test_rank_order(P, kind):
    rng = np.random.default_rng(P)
    pool = torch.empty(64 * 16, dtype=torch.uint8, device="cuda")
    rc, ctx = M.mori_create(M.mori_pool(1, 1, 1, 16, 64, pool.data_ptr()), 4096, 4096)
    assert rc == M.MORI_OK
    keep = []
    try:
        for n in (1024, P, 1024, P):
            idleness = rng.choice(np.linspace(0, 1, 97), n).astype(np.float32)  # many ties
            tier, status = rng.choice([1, 2], n).astype(np.uint8), rng.integers(0, 3, n).astype(np.uint8)
            nblk = np.zeros(n, np.int64)
            bits = idleness.view(np.uint32).astype(np.uint64)
            key = bits
            if kind != "boundary":
                nblk[tier == 2] = rng.integers(0, 9, int((tier == 2).sum()))
                if kind == "wide":
                    tier[0], status[0], nblk[0] = 2, M.MORI_ST_NEW, 1 << 19
                new = (tier == 2) & (status == M.MORI_ST_NEW)
                acting = status == M.MORI_ST_ACTING
                group = np.where(tier == 1, 1, np.where(new, 3, np.where(acting, 4, 2))).astype(np.uint64)
                sub = bits | np.where(new, nblk.astype(np.uint64) << np.uint64(30), 0).astype(np.uint64)
                sub |= np.where((tier == 1) & acting, np.uint64(1 << 31), np.uint64(0))
                key = (group << np.uint64(61)) | sub
            got = rank_order(ctx, keep, idleness, tier, status, nblk, kind != "boundary")
            log(f"rank order {kind} {n} programs")
            assert np.array_equal(got, np.argsort(key, kind="stable"))
    finally:
        torch.cuda.synchronize()
        M.mori_destroy(ctx)


@pytest.mark.parametrize("P", [1025, 1500, 4096])
def test_rejected_program(P):
    rng = np.random.default_rng(P)
    pool = torch.empty(64 * 16, dtype=torch.uint8, device="cuda")
    rc, ctx = M.mori_create(M.mori_pool(1, 1, 1, 16, 64, pool.data_ptr()), 4096, 4096)
    assert rc == M.MORI_OK
    keep = []
    try:
        idleness = rng.random(P).astype(np.float32)
        tier, status, nblk = np.full(P, 2, np.uint8), np.zeros(P, np.uint8), np.zeros(P, np.int64)
        for bad in (0, 63, 64, P - 2, P - 1):
            log(f"rejected program {bad} of {P}")
            for wrong in (2.0, np.nan):
                x = idleness.copy()
                x[bad] = wrong
                assert rank_order(ctx, keep, x, tier, status, nblk, False) == M.MORI_DEV_BAD_IDLENESS
            t = tier.copy()
            t[bad] = 9
            assert rank_order(ctx, keep, idleness, t, status, nblk, False) == M.MORI_DEV_BAD_TIER
            got = rank_order(ctx, keep, idleness, tier, status, nblk, False)
            assert np.array_equal(got, np.argsort(idleness, kind="stable"))
    finally:
        torch.cuda.synchronize()
        M.mori_destroy(ctx)


@pytest.mark.parametrize("P,k", [(256, 64), (257, 64), (1024, 16), (1024, 17), (1000, 64), (1024, 64), (1025, 64)])
def test_long_windows(orc, P, k):
    """Both sides of the line where the keys are computed by a kernel of their own."""
    rng = np.random.default_rng(P * k)
    pool = torch.empty(64 * 16, dtype=torch.uint8, device="cuda")
    rc, ctx = M.mori_create(M.mori_pool(1, 1, 1, 16, 64, pool.data_ptr()), P, 4096)
    assert rc == M.MORI_OK
    try:
        w = rng.random((P, k, 2), dtype=np.float32)
        w[rng.random(P) < 0.3] = w[0]  # ties
        rc, iota = orc.idleness(w)
        assert rc == orc.OK
        log(f"{P} programs, windows of {k}")
        dev = [torch.from_numpy(a).cuda() for a in (w, np.full(P, 2, np.uint8), np.zeros(P + 1, np.int32),
                                                    np.full(1, -1, np.int32), np.ones(64, np.uint8))]
        torch.cuda.synchronize()
        prog = M.mori_programs(P, k, dev[0].data_ptr(), None, None, dev[2].data_ptr(), 0, dev[3].data_ptr(),
                               dev[1].data_ptr(), dev[4].data_ptr())
        assert M.mori_rank_partition(ctx, prog, M.mori_budget(0, 0, 0, 0)) == M.MORI_OK
        rc, plan = M.mori_plan_wait(ctx)
        assert rc == M.MORI_OK, plan.device_error
        got = np.ctypeslib.as_array(plan.order, shape=(P,))
        assert np.array_equal(got, np.argsort(iota, kind="stable"))
    finally:
        torch.cuda.synchronize()
        M.mori_destroy(ctx)
