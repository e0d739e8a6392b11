"""Short runs over the host link: the kernel that takes the place of per-agent
copies (k_link) and the loader's unpack straight from the host copy, against the
oracle at the sizes where they can go wrong."""
import ctypes as C
import time

import numpy as np
import pytest

import workloads as W
from gpu_harness import fill_host, run_parity
from paper_2601_21473_amd import binding as B
from paper_2601_21473_amd.memory import DeviceBuffer, PoolMemory

pytestmark = pytest.mark.gpu
KIB = 1024


def ragged_trace(chunks, n_agents, max_units, seed):
    rng = np.random.default_rng(seed)
    units = rng.integers(1, max_units + 1, n_agents).astype(np.uint32)
    steps, k = 12, max(1, n_agents // 5)
    active = np.zeros((steps, n_agents), np.uint8)
    for t in range(steps):
        active[t, rng.choice(n_agents, k, replace=False)] = 1
    need = int((active.astype(np.int64) * units).sum(1).max())
    pool = W.PoolSpec("kv", need + need // 3 + 1, chunks, units)
    dist = W.exact_distances(active)
    return W.Trace("ragged", n_agents, steps, [pool], active, dist, dist.copy(), {})


@pytest.mark.parametrize("chunks,n_agents,max_units,slot_units,ring", [
    ([16], 300, 9, 4096, 2),                    # one 16-byte word a unit
    ([48, 1040, 16], 120, 5, 7, 2),             # words that fill no wave, many slots a step
    ([48, 1040, 16], 120, 5, 1, 1),             # one unit a slot, one slot
    ([4 * KIB] * 4, 200, 6, 64, 3),
    ([32 * KIB + 16], 40, 40, 50, 2),           # units longer than a round, runs over slots
    ([256 * KIB], 24, 8, 5, 2),                 # mean runs on either side of 1 MiB
])
@pytest.mark.parametrize("dirty", [False, True])
def test_short_runs(chunks, n_agents, max_units, slot_units, ring, dirty):
    tr = ragged_trace(chunks, n_agents, max_units, len(chunks) * 100 + max_units)
    mask = None
    if dirty:                                   # every other agent is written back
        mask = (np.arange(n_agents) % 2).astype(np.uint8)
        mask = np.repeat(mask[None, :], tr.n_steps, 0)
    st = run_parity(tr, theta=6, slot_units=slot_units, ring_slots=ring, dirty=mask,
                    label=f"short runs {chunks[0]}x{len(chunks)}")
    assert st["pack_launches"] > 0 and st["unpack_launches"] > 0


def test_unaligned_host_copies():
    """Host copies off the 16-byte grid keep the copies: same pool, same bytes."""
    tr = ragged_trace([4 * KIB] * 2, 60, 4, 5)
    spec, got = tr.pools[0], []
    content = W.Content(spec, seed=3)
    for shift in (0, 8):
        mem = PoolMemory(spec, 2 * 2 * 16 * spec.unit_bytes, 2)
        fill_host(mem, content, spec)
        args = mem.desc_args()
        if shift:
            mem.host_np[shift:] = mem.host_np[:-shift].copy()
            args["host_off"] = mem.host_off + np.uint64(shift)
            sizes = spec.agent_units.astype(np.int64) * spec.unit_bytes
            keep = args["host_off"].astype(np.int64) + sizes <= mem.host.nbytes
            args["host_off"][~keep] = 8         # the last agent's copy would end 8 bytes late
        pool = B.Pool(**args)
        try:
            for t in range(tr.n_steps):
                act = tr.active[t].copy()
                act[-1] = 0
                dist = np.ascontiguousarray(tr.dist[t])
                pool.plan_step(dist.ctypes.data, act.ctypes.data, 0)
                pool.evict_pack()
                pool.prefetch_unpack()
                pool.sync()
            table = pool.block_table_host_all()
            got.append((table, mem.units_bytes(table[table >= 0])))
        finally:
            pool.close()
            mem.free()
    assert np.array_equal(got[0][0], got[1][0])
    assert np.array_equal(got[0][1], got[1][1])


@pytest.mark.parametrize("shift", [0, 1])       # copies shared whole, or overlapping by half
def test_shared_host_copies(shift):
    """Victims that share a host copy write it in eviction order: the last one's
    bytes stay."""
    units = np.full(64, 2, np.uint32)
    spec = W.PoolSpec("kv", 64, [4 * KIB], units)
    mem = PoolMemory(spec, 2 * 2 * 256 * spec.unit_bytes, 2)
    content = W.Content(spec, seed=2)
    fill_host(mem, content, spec)
    start = mem.host_np.copy()
    args = mem.desc_args()
    off = np.uint64(spec.unit_bytes) * (np.uint64(shift) * (np.arange(64, dtype=np.uint64) % 8))
    args["host_off"] = off
    pool = B.Pool(**args)
    try:
        dist, act = np.full(64, 9, np.uint32), np.zeros(64, np.uint8)
        act[:32] = 1
        plans, held = [], None
        for t in range(2):                      # the first half in, then out for the second
            plans.append(pool.plan_step(dist.ctypes.data, act.ctypes.data, 0))
            pool.evict_pack()
            if t == 0:
                pool.prefetch_unpack()
                pool.sync()
                table = pool.block_table_host_all()[:64]    # units of the agents in the pool
                held = np.random.default_rng(4).integers(0, 256, (64, spec.unit_bytes), np.uint8)
                plane = np.empty_like(held)
                plane[table] = held
                mem.planes[0].upload(plane)
                act = 1 - act
        pool.sync()
        want = start.copy()
        held = held.reshape(32, -1)             # by agent
        for v in plans[1]["victims"]:
            at = int(off[v])
            want[at:at + held.shape[1]] = held[v]
        assert len(plans[1]["victims"]) == 32
        assert np.array_equal(mem.host_np, want)
    finally:
        pool.close()
        mem.free()


@pytest.mark.parametrize("chunks,slot_units", [
    ([16], 3), ([48, 1040], 5), ([64 * KIB] * 2, 16), ([64 * KIB] * 2, 17)])   # 2 MiB and above
def test_loader_chunks(chunks, slot_units):
    rng = np.random.default_rng(slot_units)
    units = rng.integers(1, 40, 12).astype(np.uint32)
    total = int(units.sum())
    spec = W.PoolSpec("kv", total, chunks, units)
    mem = PoolMemory(spec, 3 * slot_units * spec.unit_bytes, 3)
    content = W.Content(spec, seed=1)
    fill_host(mem, content, spec)
    to = rng.permutation(total).astype(np.int32)
    d_to = DeviceBuffer(to.nbytes)
    d_to.upload(to)
    off = np.concatenate([[0], np.cumsum(units.astype(np.int64))])
    loader = B.Loader([mem.desc_args()])
    try:
        loader.submit([(0, a, 5, d_to.ptr + 4 * int(off[a])) for a in range(len(units))])
        loader.pump(10_000)
        loader.sync()
        a = np.repeat(np.arange(len(units)), units)
        j = np.concatenate([np.arange(k) for k in units])
        assert np.array_equal(mem.units_bytes(to), content.units_bytes(a, j))
    finally:
        loader.close()
        d_to.free()
        mem.free()


@pytest.mark.parametrize("layout", ["one copy", "half apart", "pairs"])
@pytest.mark.parametrize("loads", [False, True])
def test_shared_host_copies_direct(layout, loads):
    """Direct steps: victims that share a host copy write it in eviction order,
    and the step's loads read it after them.  The copies: one for all agents;
    four, each overlapping the next by half; one for every two agents, so that
    only a victim and a load share."""
    n, s = 256, 2
    units = np.full(n, s, np.uint32)
    spec = W.PoolSpec("kv", n, [4 * KIB], units)
    size = s * spec.unit_bytes
    mem = PoolMemory(spec, 2 * 2 * n * spec.unit_bytes, 2)
    fill_host(mem, W.Content(spec, seed=2), spec)
    want = mem.host_np.copy()
    args = mem.desc_args()
    a = np.arange(n, dtype=np.uint64)
    args["host_off"] = {"one copy": a * 0, "half apart": a % 4 * np.uint64(size // 2),
                        "pairs": a % (n // 2) * np.uint64(size)}[layout]
    off = args["host_off"].astype(np.int64)
    pool = B.Pool(**args, direct_bytes=4 << 20)
    try:
        act = np.zeros((2, n), np.uint8)
        act[0, :n // 2] = 1                     # the first half in, then out for the second
        act[1, n // 2:] = 1
        dist = np.full(n, 9, np.uint32)
        pool.plan_step(dist.ctypes.data, act[0].ctypes.data, 0)
        pool.evict_pack()
        pool.prefetch_unpack()
        pool.sync()
        table = pool.block_table_host_all().reshape(n, s)
        held = np.random.default_rng(4).integers(0, 256, (n, spec.unit_bytes), np.uint8)
        mem.planes[0].upload(held)
        plan = pool.plan_step(dist.ctypes.data, act[1].ctypes.data, 0)
        assert len(plan["victims"]) == n // 2 and len(plan["loads"]) == n // 2
        pool.evict_pack()
        if loads:
            pool.prefetch_unpack()
        pool.sync()
        for v in plan["victims"]:
            want[off[v]:off[v] + size] = held[table[v]].reshape(-1)
        assert np.array_equal(mem.host_np, want)
        if not loads:
            return
        table = pool.block_table_host_all().reshape(n, s)
        got = mem.units_bytes(table[plan["loads"]].reshape(-1)).reshape(-1, size)
        exp = np.stack([want[off[b]:off[b] + size] for b in plan["loads"]])
        assert np.array_equal(got, exp)
    finally:
        pool.close()
        mem.free()


def device_free():
    """Bytes free on the device, from the HIP runtime that the library runs on."""
    hip = C.CDLL("libamdhip64.so")
    free, total = C.c_size_t(), C.c_size_t()
    assert hip.hipMemGetInfo(C.byref(free), C.byref(total)) == 0
    return free.value


@pytest.mark.parametrize("form,lists", [("short", True), ("long", False), ("unaligned", False)])
def test_offset_lists_only_where_they_serve(form, lists):
    """Host-copy offsets (16 bytes a unit) are kept on the device only by pools
    whose steps can go by k_link: not if every agent has more than 1 MiB, nor with
    copies off the 16-byte grid."""
    capacity = 8 << 20
    units = np.full(4, (1 << 16) + (form == "long"), np.uint32)
    spec = W.PoolSpec("kv", capacity, [16], units)
    mem = PoolMemory(spec, 2 * 1024 * 16, 1)
    args = mem.desc_args()
    if form == "unaligned":
        args["host_off"] = mem.host_off + np.uint64(8)
        args["host_off"][-1] -= np.uint64(8)
    try:
        B.Pool(**args).close()                  # the shared streams and their memory
        before = device_free()
        pool = B.Pool(**args)
        used = before - device_free()
        pool.close()
        plain = 4 * 4 * capacity                # the plan's unit lists, whatever the form
        assert used >= plain + 16 * capacity if lists else used < plain + 8 * capacity, used
    finally:
        mem.free()


@pytest.mark.parametrize("chunks,slot_units", [
    ([16] * 256, 16), ([16] * 256, 17), ([256] * 256, 17), ([240] * 256, 17)])
def test_loader_chunks_of_small_planes(chunks, slot_units):
    """4,096 pieces a chunk and more, of 256 bytes and less."""
    test_loader_chunks(chunks, slot_units)


def test_loader_time_of_tiny_planes():
    """Chunks of many tiny planes take no longer than copied ones, which chunks
    off the 16-byte grid always are (by reads over the link they took 2.6 times as
    long)."""
    units, slot_units = np.full(4, 4096, np.uint32), 256
    spec = W.PoolSpec("kv", int(units.sum()), [16] * 64, units)
    mem = PoolMemory(spec, 2 * 4 * slot_units * spec.unit_bytes, 4)
    mem.host_np[:] = 1
    to = np.random.default_rng(0).permutation(int(units.sum())).astype(np.int32)
    d_to = DeviceBuffer(to.nbytes)
    d_to.upload(to)
    ms = []
    try:
        for shift in (0, 8):
            args = mem.desc_args()
            args["host_off"] = mem.host_off + np.uint64(shift)
            args["host_off"][-1] = 0
            loader = B.Loader([args])
            times = []
            for _ in range(5):
                loader.sync()
                t0 = time.perf_counter()
                loader.submit([(0, a, 5, d_to.ptr + 4 * 4096 * a) for a in range(3)])
                loader.pump(10_000)
                loader.sync()
                times.append(time.perf_counter() - t0)
            loader.close()
            ms.append(1e3 * min(times))
        print(f"[loader] tiny planes {ms[0]:.2f} ms, copied {ms[1]:.2f} ms", flush=True)
        assert ms[0] <= 1.5 * ms[1]
    finally:
        d_to.free()
        mem.free()
