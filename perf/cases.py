"""Performance cases of libmori: what a serving system has it do.

Five kinds of work, each through the public entry points.  Every pass can be
repeated on its state: a placement pass is a pair of plans (there and back), so
that each pass starts from the tiers the one before left.

  plan   mori_rank_partition + mori_plan_wait, two plans a pass under alternating
         windows and budgets; placement only, as a router's scheduler tick.
  evict  mori_evict_order (or its allocation-free form) over the block metadata
         of one tier, as the engine does before it allocates.
  swap   plan + mori_kv_swap_out + mori_kv_swap_in with the lower tier's buffers
         in registered device memory, nothing blocking the host: the gather and
         scatter kernels without the host link.
  step   tiering.TierPool.step with the lower tier in pinned host memory, two
         synchronous rebalances a pass: what a serving loop calls.
  admit  mori_replica_admit, host code of the router.

All outputs are whole numbers or bytes and are the same for every correct
implementation, so the tolerance is "exact" throughout.
"""
from __future__ import annotations

import ctypes
import math

import numpy as np
import torch

from paper_2606_00866_amd import mori as M
from paper_2606_00866_amd.tiering import TierPool, check

MIB = 1 << 20
POLICIES = {  # name: flags
    "boundary": 0,
    "status": M.MORI_F_STATUS_KEY,
    "skip_fit": M.MORI_F_SKIP_FIT,
    "ssd": M.MORI_F_SSD_TIER,
    "ssd_status": M.MORI_F_SSD_TIER | M.MORI_F_STATUS_KEY,
    "incremental": M.MORI_F_INCREMENTAL,
    "incremental_skip": M.MORI_F_INCREMENTAL | M.MORI_F_SKIP_FIT,
}
WINDOW_KS = (1, 5, 5, 5, 16, 64)


def listed():
    return [
        # the smallest deployment: a handful of agents on one small pool, latency only
        {"name": "plan_8", "kind": "plan", "programs": 8, "pages": 536, "window": 5, "policy": "boundary",
         "gpu": 0.6, "cpu": 0.3, "pool": 1.0},
        # the compressed-latent workload's programs and pages at a scheduler tick
        {"name": "plan_256", "kind": "plan", "programs": 256, "pages": 37103, "window": 5, "policy": "boundary",
         "gpu": 0.4, "cpu": 0.2, "pool": 1.0},
        # many short sessions in a tight pool under the paper's incremental policy
        {"name": "plan_1024_incremental", "kind": "plan", "programs": 1024, "pages": 150001, "window": 5,
         "policy": "incremental_skip", "gpu": 0.55, "cpu": 0.3, "pool": 0.65},
        # the most programs a context takes, three tiers, statuses in the key
        {"name": "plan_4096_ssd", "kind": "plan", "programs": 4096, "pages": 400003, "window": 5,
         "policy": "ssd_status", "gpu": 0.5, "cpu": 0.25, "pool": 0.75},
        # one tier's eviction order: a small tier from a capturing serving loop,
        # one Llama-3-8B pool's pages, and radix-tree nodes of a large host tier
        {"name": "evict_4096", "kind": "evict", "blocks": 4096, "programs": 64, "ties": 0.5, "sizes": False,
         "tier": 0, "horizon_bits": 40, "noalloc": True},
        {"name": "evict_69938", "kind": "evict", "blocks": 69938, "programs": 1024, "ties": 0.5, "sizes": True,
         "tier": 0, "horizon_bits": 40, "noalloc": False},
        {"name": "evict_1048576", "kind": "evict", "blocks": 1 << 20, "programs": 1024, "ties": 0.5, "sizes": True,
         "tier": 1, "horizon_bits": 40, "noalloc": False},
        # gather and scatter over HBM: 72 KiB compressed-latent runs, and the 4 KiB
        # runs of one rank at tensor parallelism 8
        {"name": "swap_72k", "kind": "swap", "programs": 64, "mib": 6144, "planes": 61, "tokens": 64, "row": 1152,
         "pool": 1.0},
        {"name": "swap_4k", "kind": "swap", "programs": 64, "mib": 1536, "planes": 160, "tokens": 16, "row": 256,
         "pool": 0.65},
        # whole rebalances over the host link: the tiny workload, and 32 KiB
        # Llama-3-8B runs at a size where the link decides
        {"name": "step_tiny", "kind": "step", "programs": 8, "mib": 17, "planes": 4, "tokens": 16, "row": 512,
         "pool": 1.0, "mode": 0},
        {"name": "step_32k", "kind": "step", "programs": 32, "mib": 1024, "planes": 64, "tokens": 16, "row": 2048,
         "pool": 1.0, "mode": 0},
        # the router's shared Waiting queue over the replicas of a cluster
        {"name": "admit_4096", "kind": "admit", "programs": 4096, "replicas": 64, "best_fit": False},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["plan"] * 4 + ["evict"] * 4 + ["swap"] * 2 + ["step"] * 2 + ["admit"])
    if kind == "plan":
        programs = _log_int(rng, 8, 4096)
        return {"kind": "plan", "programs": programs, "pages": _log_int(rng, 4 * programs, min(400000, 400 * programs)),
                "window": rng.choice(WINDOW_KS), "policy": rng.choice(sorted(POLICIES)),
                "gpu": round(rng.uniform(0.35, 0.55), 3), "cpu": round(rng.uniform(0.2, 0.4), 3),
                "pool": round(rng.uniform(0.7, 1.0), 3)}
    if kind == "evict":
        blocks = _log_int(rng, 256, 1 << 20)
        return {"kind": "evict", "blocks": blocks, "programs": _log_int(rng, 8, 1024), "ties": round(rng.random(), 3),
                "sizes": rng.random() < 0.6, "tier": rng.randrange(2), "horizon_bits": rng.choice([32, 40, 50]),
                "noalloc": blocks <= M.MORI_EVICT_NOALLOC_MAX_BLOCKS and rng.random() < 0.4}
    if kind == "admit":
        return {"kind": "admit", "programs": _log_int(rng, 64, 4096), "replicas": _log_int(rng, 2, 64),
                "best_fit": rng.random() < 0.5}
    tokens = rng.choice([16, 16, 32, 64])
    row = rng.choice([256, 512, 656, 1024, 1152, 2048])
    planes = rng.choice([4, 32, 61, 64, 160])
    mib = _log_int(rng, 32, 4096 if kind == "swap" else 1024)
    most = max(2, mib * MIB // (planes * tokens * row) // 2)  # at least two blocks a program
    case = {"kind": kind, "programs": min(_log_int(rng, 8, 256), most), "mib": mib, "planes": planes,
            "tokens": tokens, "row": row, "pool": round(rng.uniform(0.65, 1.0), 3)}
    if kind == "step":
        case["mode"] = rng.choice([M.MORI_COPY_AUTO, M.MORI_COPY_AUTO, M.MORI_COPY_KERNEL])
    return case


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------
class State:
    """What a pass works on."""

    def __init__(self, case, seed):
        self.case = case
        self.rng = np.random.default_rng([seed, 0x6D6F7269])


class Owner:
    """Closes a context or a TierPool once neither a state nor a view of its host memory needs it."""

    def __init__(self, close, arg):
        self.close, self.arg = close, arg

    def __del__(self):
        self.close(self.arg)

    def view(self, addr, n, dtype):
        """numpy view of n values at a host address, which keeps the owner alive."""
        return np.asarray(_View(self, addr, n, np.dtype(dtype)))


class _View:
    def __init__(self, owner, addr, n, dtype):
        self.owner = owner
        self.__array_interface__ = {"shape": (n,), "typestr": dtype.str, "data": (addr, False), "version": 3}


_STREAMS = []


def _streams():
    """The program's swap-out and swap-in streams, created once."""
    if not _STREAMS:
        _STREAMS.extend([torch.cuda.Stream(), torch.cuda.Stream()])
    return _STREAMS


def _windows(rng, busy, k):
    """[P][k][2] seconds: reasoning about 2 s; tool calls about 1 s (busy) or
    60 s (idle); the newest tool call is still running."""
    P = busy.size
    r = np.exp(math.log(2.0) + 0.5 * rng.standard_normal((P, k)))
    a = np.exp(np.where(busy, 0.0, math.log(60.0))[:, None] + rng.standard_normal((P, k)))
    a[:, -1] *= rng.random(P)
    return np.stack([r, a], axis=2).astype(np.float32)


def _block_counts(rng, P, total):
    """P positive block counts with lognormal spread that sum to about total (exactly, for total >= P)."""
    w = np.exp(0.5 * rng.standard_normal(P))
    n = np.maximum(1, np.floor(w / w.sum() * total)).astype(np.int64)
    n[int(np.argmax(n))] += max(0, total - int(n.sum()))
    return n


def _chunked_pages(rng, NB):
    """All page ids in an order of chunks of mean 4 consecutive pages (a used pool)."""
    lens = rng.geometric(0.25, size=NB)
    cuts = np.cumsum(lens)
    cuts = np.concatenate([[0], cuts[cuts < NB], [NB]])
    order = rng.permutation(cuts.size - 1)
    starts, ends = cuts[:-1][order], cuts[1:][order]
    n = ends - starts
    base = np.repeat(starts - np.concatenate([[0], np.cumsum(n)[:-1]]), n)
    return (base + np.arange(NB)).astype(np.uint32)


def _tables(rng, nblk, tier, NB):
    off = np.zeros(nblk.size + 1, np.uint32)
    off[1:] = np.cumsum(nblk)
    tbl = np.full(int(off[-1]), M.MORI_NO_PAGE, np.uint32)
    pages = _chunked_pages(rng, NB)
    used = 0
    for p in np.flatnonzero(tier == M.MORI_TIER_GPU):
        n = int(nblk[p])
        tbl[off[p]:off[p] + n] = pages[used:used + n]
        used += n
    free = np.zeros(NB, np.uint8)
    free[pages[used:]] = 1
    return off, tbl, free


def _dev(a):
    a = np.ascontiguousarray(a)
    if a.dtype == np.uint32:
        a = a.view(np.int32)
    return torch.from_numpy(a.copy()).cuda()


def _fill(nbytes, seed):
    """Random bytes on the device (KV values)."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.randint(-(1 << 62), 1 << 62, (nbytes // 8,), dtype=torch.int64, device="cuda", generator=g)


def _there_and_back(rng, P, k=5):
    """Half of the programs busy, then the other half: (first half's ids, windows there, windows back)."""
    first = np.zeros(P, bool)
    first[rng.permutation(P)[: P // 2]] = True
    lo = lambda m: np.stack([rng.uniform(1.5, 2.5, (P, k)),
                             np.where(m[:, None], rng.uniform(0, 0.3, (P, k)), rng.uniform(40, 80, (P, k)))],
                            axis=2).astype(np.float32)
    return first, lo(first), lo(~first)


def _prepare_plan(st, case, seed):
    rng, P = st.rng, case["programs"]
    nblk = _block_counts(rng, P, case["pages"])
    total = int(nblk.sum())
    NB = max(1, math.ceil(case["pool"] * total))
    flags = POLICIES[case["policy"]]
    st.block = 16
    # tiers of a running system: filled in id order within the budgets
    gpu, cpu = int(min(case["gpu"], case["pool"]) * total), int(case["cpu"] * total)
    cum = np.cumsum(nblk)
    tier = np.full(P, M.MORI_TIER_WAIT, np.uint8)
    tier[cum <= gpu] = M.MORI_TIER_GPU
    n_gpu = int((cum <= gpu).sum())
    base = int(cum[n_gpu - 1]) if n_gpu else 0
    tier[(cum > gpu) & (cum - base <= cpu)] = M.MORI_TIER_CPU
    off, tbl, free = _tables(rng, nblk, tier, NB)
    busy = rng.random(P) < 0.5
    flip = busy ^ (rng.random(P) < 0.1)
    st.keep = []
    st.calls = []
    pool = torch.empty(NB * st.block, dtype=torch.uint8, device="cuda")
    st.tbl, st.tier, st.free = _dev(tbl), _dev(tier), _dev(free)
    d_off = _dev(off)
    st.keep += [pool, d_off]
    for b, swing in ((busy, 0.9), (flip, 1.1)):
        w = _dev(_windows(rng, b, case["window"]))
        status = _dev(np.where(rng.random(P) < 0.1, M.MORI_ST_NEW, np.where(b, M.MORI_ST_REASONING, M.MORI_ST_ACTING))
                      .astype(np.uint8))
        st.keep += [w, status]
        prog = M.mori_programs(P, case["window"], w.data_ptr(), None, status.data_ptr(), d_off.data_ptr(), total,
                               st.tbl.data_ptr(), st.tier.data_ptr(), st.free.data_ptr())
        budget = M.mori_budget(min(NB, int(gpu * swing)) * st.block, cpu * st.block, flags, int(0.1 * total) * st.block)
        st.calls.append((prog, budget))
    desc = M.mori_pool(1, 1, 1, st.block, NB, pool.data_ptr())
    rc, st.ctx = M.mori_create(desc, P, 4096)
    check(rc, "mori_create")
    st.owner = Owner(M.mori_destroy, st.ctx)
    st.stream = _streams()[0].cuda_stream
    st.views = None


def _plan_views(owner, plan):
    """The plan's arrays in the context's pinned mirror (as numpy views)."""
    view = lambda ptr, dtype: owner.view(ctypes.addressof(ptr.contents), plan.num_programs, dtype)
    return {"order": view(plan.order, np.uint32), "prefix": view(plan.prefix, np.uint64),
            "tier_new": view(plan.tier_new, np.uint8), "category": view(plan.category, np.uint8)}


def _run_plan(st):
    for prog, budget in st.calls:
        check(M.mori_rank_partition(st.ctx, prog, budget, st.stream), "mori_rank_partition")
        rc, plan = M.mori_plan_wait(st.ctx)
        check(rc, "mori_plan_wait")
    if st.views is None:  # the mirror stays where it is for the life of the context
        st.views = _plan_views(st.owner, plan)
    return {"tbl": st.tbl, "tier": st.tier, "free": st.free, **st.views,
            "counts": [plan.m_gpu, plan.m_cpu, plan.m_ssd, plan.n_out, plan.n_in, plan.pages_out, plan.pages_in,
                       plan.pages_admit, plan.pages_free_after, plan.gpu_bytes_after]}


def _geometry(case):
    run = case["tokens"] * case["row"]
    block = case["planes"] * run
    total = max(2 * case["programs"], case["mib"] * MIB // block)
    return run, block, total


def _tier_split(st, case):
    """Programs, tables and windows of a there-and-back rebalance: the second half starts on the GPU."""
    rng, P = st.rng, case["programs"]
    run, block, total = _geometry(case)
    nblk = _block_counts(rng, P, total)
    first, w_there, w_back = _there_and_back(rng, P)
    a, b = int(nblk[first].sum()), int(nblk[~first].sum())
    gpu = max(a, b)
    NB = max(gpu, math.ceil(case["pool"] * int(nblk.sum())))
    tier = np.where(first, M.MORI_TIER_CPU, M.MORI_TIER_GPU).astype(np.uint8)
    off, tbl, free = _tables(rng, nblk, tier, NB)
    return run, block, nblk, first, (w_there, w_back), gpu, NB, tier, off, tbl, free


def _prepare_swap(st, case, seed):
    run, block, nblk, first, wins, gpu, NB, tier, off, tbl, free = _tier_split(st, case)
    P, total = nblk.size, int(nblk.sum())
    st.pool = _fill(NB * block, seed)
    st.lower = _fill(total * block, seed + 1)
    st.addr = (st.lower.data_ptr() + off[:-1].astype(np.uint64) * np.uint64(block)).astype(np.uint64)
    st.tbl, st.tier, st.free = _dev(tbl), _dev(tier), _dev(free)
    d_off = _dev(off)
    st.keep = [d_off]
    st.calls = []
    for w in wins:
        w = _dev(w)
        st.keep.append(w)
        st.calls.append((M.mori_programs(P, 5, w.data_ptr(), None, None, d_off.data_ptr(), total, st.tbl.data_ptr(),
                                         st.tier.data_ptr(), st.free.data_ptr()),
                         M.mori_budget(gpu * block, total * block, 0, 0)))
    desc = M.mori_pool(case["planes"], 1, case["tokens"], case["row"], NB, st.pool.data_ptr())
    rc, st.ctx = M.mori_create(desc, P, 2 * run)
    check(rc, "mori_create")
    st.owner = Owner(M.mori_destroy, st.ctx)
    check(M.mori_register(st.ctx, st.lower.data_ptr(), st.lower.numel() * 8), "mori_register")
    st.s_out, st.s_in = (s.cuda_stream for s in _streams())


def _run_swap(st):
    addr = st.addr.ctypes.data
    for prog, budget in st.calls:
        check(M.mori_rank_partition(st.ctx, prog, budget, st.s_out), "mori_rank_partition")
        check(M.mori_kv_swap_out(st.ctx, addr, M.MORI_COPY_AUTO, st.s_out), "mori_kv_swap_out")
        check(M.mori_kv_swap_in(st.ctx, addr, M.MORI_COPY_AUTO, st.s_in), "mori_kv_swap_in")
    return {"pool": st.pool, "lower": st.lower, "tbl": st.tbl, "tier": st.tier, "free": st.free}


class _Geom:
    def __init__(self, case, NB):
        self.layers, self.planes = case["planes"], 1
        self.block_tokens, self.row_bytes, self.num_blocks = case["tokens"], case["row"], NB


def _prepare_step(st, case, seed):
    run, block, nblk, first, wins, gpu, NB, tier, off, tbl, free = _tier_split(st, case)
    total = int(nblk.sum())
    arena = (total + total // 2 + 2) * block + 4096 * (nblk.size + 1)  # first-fit extents need room to spare
    st.tp = TierPool(_Geom(case, NB), off, tbl, tier, free, arena_bytes=arena + -arena % 4096,
                     pool=_fill(NB * block, seed).view(torch.uint8))
    st.owner = Owner(TierPool.close, st.tp)
    st.arena = st.owner.view(st.tp.arena.ptr, st.tp.arena.nbytes // 8, np.int64)
    part = _fill(8 << 20, seed + 1).cpu().numpy()
    for at in range(0, st.arena.size, part.size):
        st.arena[at:at + part.size] = part[: st.arena.size - at]
    for p in np.flatnonzero(first):
        st.tp.give_host_buffer(int(p))
    st.wins = [_dev(w) for w in wins]
    st.gpu_bytes, st.cpu_bytes = gpu * block, total * block
    st.streams = _streams()


def _run_step(st):
    s_out, s_in = st.streams
    for w in st.wins:
        st.tp.step(gpu_bytes=st.gpu_bytes, cpu_bytes=st.cpu_bytes, window=w, mode=st.case["mode"], s_out=s_out,
                   s_in=s_in)
    return {"pool": st.tp.pool.view(torch.int64), "arena": st.arena, "tbl": st.tp.tbl, "tier": st.tp.tier,
            "free": st.tp.free_map}


def _prepare_evict(st, case, seed):
    """Blocks dealt to programs in contiguous runs; a share of the programs stamp
    all their blocks with one time, the others' blocks are older by a random step."""
    rng, N = st.rng, case["blocks"]
    P = min(case["programs"], N)
    cuts = np.sort(rng.choice(np.arange(1, N), size=P - 1, replace=False)) if N > 1 else np.zeros(0, np.int64)
    owner = np.zeros(N, np.int64)
    owner[cuts] = 1
    owner = np.cumsum(owner)
    ptype = rng.choice(3, size=P, p=[0.5, 0.3, 0.2]).astype(np.uint8)
    ptime = rng.integers(0, 1 << case["horizon_bits"], size=P)
    tied = rng.random(P) < case["ties"]
    t = np.clip(ptime[owner] - np.where(tied[owner], 0, rng.integers(1, 1 << 20, size=N)), 0, None)
    size = rng.integers(1, 17, size=N).astype(np.uint32) if case["sizes"] else None
    d_type, d_time = _dev(ptype[owner]), _dev(t.astype(np.int64))
    d_size = None if size is None else _dev(size)
    units = N if size is None else int(size.astype(np.int64).sum())
    st.need = units * 4096 // 4
    rc, st.ws_bytes = M.mori_evict_workspace(N)
    check(rc, "mori_evict_workspace")
    st.ws = None if case["noalloc"] else torch.empty(st.ws_bytes, dtype=torch.uint8, device="cuda")
    st.order = torch.empty(N, dtype=torch.int32, device="cuda")
    st.prefix = torch.empty(N, dtype=torch.int64, device="cuda")
    st.result = torch.zeros(2, dtype=torch.int32, device="cuda")
    st.keep = [d_type, d_time, d_size]
    st.blk = M.mori_blocks(N, d_type.data_ptr(), d_time.data_ptr(), None if d_size is None else d_size.data_ptr(),
                           4096)


def _run_evict(st):
    s = torch.cuda.current_stream().cuda_stream
    out = (st.order.data_ptr(), st.prefix.data_ptr(), st.result.data_ptr(), s)
    if st.ws is None:
        check(M.mori_evict_order_noalloc(st.blk, st.case["tier"], st.need, *out), "mori_evict_order_noalloc")
    else:
        check(M.mori_evict_order(st.blk, st.case["tier"], st.need, st.ws.data_ptr(), st.ws_bytes, *out),
              "mori_evict_order")
    return {"order": st.order, "prefix": st.prefix, "result": st.result}


def _prepare_admit(st, case, seed):
    rng, P, R = st.rng, case["programs"], case["replicas"]
    st.bytes = (rng.lognormal(math.log(2 << 30), 0.8, size=P) // 16 * 16).astype(np.uint64)
    st.idleness = rng.random(P).astype(np.float32)
    st.status = rng.choice(3, size=P, p=[0.4, 0.3, 0.3]).astype(np.uint8)
    st.room = rng.integers(0, 64 << 30, size=R).astype(np.uint64)
    st.flags = M.MORI_ADMIT_BEST_FIT if case["best_fit"] else 0


def _run_admit(st):
    rc, replica, room_after = M.mori_replica_admit(st.bytes, st.idleness, st.status, st.room, st.flags)
    check(rc, "mori_replica_admit")
    return {"replica": replica, "room_after": room_after.view(np.int64)}


_PREPARE = {"plan": _prepare_plan, "evict": _prepare_evict, "swap": _prepare_swap, "step": _prepare_step,
            "admit": _prepare_admit}
_RUN = {"plan": _run_plan, "evict": _run_evict, "swap": _run_swap, "step": _run_step, "admit": _run_admit}


def prepare(case, seed):
    st = State(case, seed)
    _PREPARE[case["kind"]](st, case, seed)
    return st


def run(state):
    return _RUN[state.case["kind"]](state)


def work(case):
    """Bytes of one pass: every input read once, every output written once."""
    kind = case["kind"]
    if kind == "plan":  # two plans: windows, offsets, tables and free map in; plan, changed tables, tiers, map out
        P, E = case["programs"], case["pages"]
        NB = math.ceil(case["pool"] * E)
        one = P * (8 * case["window"] + 4 + 1 + 1) + 4 * E + NB + P * (4 + 8 + 3) + 4 * E // 4 + NB
        return {"bytes": 2 * one, "flops": 2 * P * 2 * case["window"]}
    if kind == "evict":  # type, time, size in; order and prefix out
        return {"bytes": case["blocks"] * (1 + 8 + (4 if case["sizes"] else 0) + 4 + 8), "flops": 0}
    if kind == "admit":
        return {"bytes": case["programs"] * (8 + 4 + 1 + 4) + 16 * case["replicas"], "flops": 0}
    run_, block, total = _geometry(case)
    # two rebalances, each moving about half of the KV out and half in: read and written once
    return {"bytes": 2 * total * block * 2, "flops": 0}


def tolerance(case):
    return "exact"
