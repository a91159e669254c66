"""Swaps at the edges of the copy shapes and of the unit decode:
runs on both sides of every shape's limit, and hundreds of programs of zero to
three blocks, so that a grid stride passes many programs and both parts of a
swap-in begin and end inside the list.  Kernel-direct with buffers in registered
device memory and in pinned host memory, and through staging; every resident
byte against the oracle."""
import numpy as np
import pytest
import torch

from gpu_helpers import log
from oracle import oracle
from paper_2606_00866_amd import mori as M
from paper_2606_00866_amd.tiering import TierPool
from workload import Geometry, fill_pool_np, make_bank, program_host_content, random_instance

pytestmark = pytest.mark.gpu

# vectors of 16 B per run: 64 | 65, 128 | 129, 256 (even) and 257, 656, 1023 | 1024 | 1025, 2047 | 2048, 4608
VECTORS = [1, 64, 65, 128, 129, 256, 257, 656, 1023, 1024, 1025, 2047, 2048, 4608]


@pytest.mark.parametrize("where", ["device", "host", "staging"])
@pytest.mark.parametrize("vectors", VECTORS)
def test_many_small_programs(vectors, where):
    mode = M.MORI_COPY_CE if where == "staging" else M.MORI_COPY_KERNEL
    rng = np.random.default_rng(vectors)
    geom = Geometry(layers=3, planes=1, block_tokens=1, row_bytes=16 * vectors, num_blocks=0)
    inst = random_instance(rng, P=300 if vectors < 1000 else 80, max_blocks=3, geom=geom, tier_p=(0.55, 0.45),
                           extra_free=5)
    g, bb = inst.geom, inst.geom.block_bytes
    bank = make_bank(3, inst.dtype, g.run_bytes)
    pool = fill_pool_np(inst, bank)
    bufs = [program_host_content(inst, bank, p).copy() if inst.tier[p] == 1
            else np.zeros(int(inst.nblk[p]) * bb, np.uint8) for p in range(inst.P)]
    off = inst.tbl_off.astype(np.int64) * bb
    lower = np.concatenate(bufs)
    tbl, tier, free = inst.copy_state()
    tp = TierPool(g, inst.tbl_off, inst.tbl, inst.tier, inst.free_map, arena_bytes=lower.size + 4096)
    try:
        tp.pool.copy_(torch.from_numpy(pool).cuda())
        if where == "device":
            dbuf = torch.from_numpy(lower).cuda()
            assert M.mori_register(tp.ctx, dbuf.data_ptr(), dbuf.numel()) == M.MORI_OK
            base, read = dbuf.data_ptr(), lambda: dbuf.cpu().numpy()
        else:
            tp.arena.view(tp.arena.ptr, lower.size)[:] = lower
            base, read = tp.arena.ptr, lambda: tp.arena.view(tp.arena.ptr, lower.size).copy()
        addr = np.array([base + int(o) for o in off[:-1]], np.uint64)
        s_out, s_in = torch.cuda.Stream(), torch.cuda.Stream()
        for t in range(3):
            w = np.ascontiguousarray(inst.window if t != 1 else inst.window[:, :, ::-1])
            bg = (int(0.7 * g.num_blocks) if t != 2 else g.num_blocks) * bb
            res = oracle.rebalance(g, window=w, tbl_off=inst.tbl_off, tbl=tbl, tier=tier, free_map=free,
                                   gpu_budget=bg, cpu_budget=inst.total_bytes, pool=pool, host_bufs=bufs)
            assert res.rc == oracle.OK
            assert tp.rank_partition(gpu_bytes=bg, cpu_bytes=inst.total_bytes, window=torch.from_numpy(w).cuda(),
                                     stream=s_out) == 0
            assert M.mori_kv_swap_out(tp.ctx, addr.ctypes.data, mode, s_out.cuda_stream) == M.MORI_OK
            assert M.mori_kv_swap_in(tp.ctx, addr.ctypes.data, mode, s_in.cuda_stream) == M.MORI_OK
            torch.cuda.synchronize()
            assert M.mori_query(tp.ctx, M.MORI_Q_DEVICE_ERROR) == (M.MORI_OK, 0)
            rc, plan = tp.plan_wait()
            log(f"  {where} {vectors} vectors step {t}: out {plan.n_out} in {plan.n_in} recycled {plan.pages_recycled}")
            t_, r_, f_ = tp.state()
            assert (t_ == tbl).all() and (r_ == tier).all() and (f_ == free).all()
            owned = tbl[tbl != 0xFFFFFFFF].astype(np.int64)
            dpool = tp.pool.cpu().numpy().reshape(g.nplanes, g.num_blocks, g.run_bytes)
            assert np.array_equal(dpool[:, owned], pool.reshape(g.nplanes, g.num_blocks, g.run_bytes)[:, owned])
            low = read()
            for p in np.flatnonzero(tier == 1):
                assert np.array_equal(low[off[p]:off[p + 1]], bufs[p]), p
    finally:
        torch.cuda.synchronize()
        tp.close()
