"""Measured cases: what a program built on this framework asks of it.

Five kinds of work, each through the public binding
(``paper_2601_21473_amd.binding``):

``step``         simulation steps of a memory pool: ``plan_step`` ->
                 ``evict_pack`` -> ``prefetch_unpack`` on one stream, from a
                 64-agent pool whose step is all latency to adapter pools whose
                 step is all host link; a pass is one step, or one period of
                 the schedule where the steps differ much in what they move;
``loader``       the load-task scheduler: background loads, an urgent task that
                 interrupts them, everything pumped to the end;
``objects``      distances and activity of shared memory objects from those of
                 the agents that reference them;
``hops``         hop counts from the active agents over a message graph;
``interaction``  distances from the nearest other agent on a tile grid.

Every output is a whole number or a byte that was moved, so two correct
implementations agree exactly and there is nothing to compare in 64 bits.
"""
import math

import numpy as np
import torch

from paper_2601_21473_amd import binding

KIB, MIB = 1 << 10, 1 << 20
NEVER = 0xFFFFFFFF


def listed():
    return [
        # The smallest call: 64 agents of 16 pages (2-layer, 2-head, 64-wide
        # fp16 KV, 4 planes of 4 KiB), pool of 16 agents, 6 active per step,
        # exact distances.  A step is launches and host work.
        dict(name="step_64", kind="step", agents=64, units_lo=16, units_hi=16, planes=4,
             chunk=4 * KIB, capacity=256, active=6, period=32, steps=1, noise=0, threshold=NEVER,
             budget=0, inputs="device", dirty="all", shared=0, direct=4 * MIB, slot_units=256, ring=4),
        # Prefix KV of a large model (32 layers x 8 heads x 128 bf16: 64 planes
        # of 32 KiB, 2 MiB a page), ragged agents: the host link is the bound.
        dict(name="step_kv_pages", kind="step", agents=48, units_lo=8, units_hi=32, planes=64,
             chunk=32 * KIB, capacity=300, active=5, period=16, steps=16, noise=0, threshold=NEVER,
             budget=0, inputs="device", dirty="all", shared=0, direct=4 * MIB, slot_units=32, ring=4),
        # Read-only adapters (80 MiB each in 448 planes): many agents behind 16
        # host copies, nothing to write back, loads only.
        dict(name="step_adapters", kind="step", agents=2000, units_lo=1, units_hi=1, planes=448,
             chunk=187232, capacity=64, active=16, period=8, steps=8, noise=0, threshold=6,
             budget=16, inputs="device", dirty="none", shared=16, direct=0, slot_units=4, ring=4),
        # Ten thousand small agents in bursts with noisy distances, memory of a
        # small model: hundreds of small moves per step in both directions.
        dict(name="step_10k_bursty", kind="step", agents=10_000, units_lo=1, units_hi=11, planes=4,
             chunk=4 * KIB, capacity=15_000, active=240, period=32, steps=32, noise=2, threshold=4,
             budget=0, inputs="device", dirty="all", shared=0, direct=4 * MIB, slot_units=1024, ring=4),
        # Fifty thousand agents, a quiet step (few active, a small prefetch
        # budget), host arrays in, half of the agents' memory unchanged.
        dict(name="step_50k_quiet", kind="step", agents=50_000, units_lo=1, units_hi=3, planes=1,
             chunk=16 * KIB, capacity=4_000, active=60, period=64, steps=1, noise=2, threshold=8,
             budget=48, inputs="host", dirty="half", shared=0, direct=4 * MIB, slot_units=1024, ring=4),
        # The load scheduler on large-model pages, 32 MiB chunks.
        dict(name="loader_kv", kind="loader", agents=40, units_lo=8, units_hi=32, planes=64,
             chunk=32 * KIB, urgent=4, slot_units=16, ring=4),
        # Shared prefix trees: one simulation, and many side by side.
        dict(name="objects_16k", kind="objects", trees=1, agents=16_384, branching=8, depth=5,
             active=0.01),
        dict(name="objects_forest", kind="objects", trees=160, agents=50_000, branching=8, depth=5,
             active=0.01),
        # Information diffusion: out-degree-8 message graphs, 1% of the agents
        # hold the information.
        dict(name="hops_50k", kind="hops", vertices=50_000, degree=8, skew=False, sources=500,
             max_hops=NEVER),
        dict(name="hops_4m", kind="hops", vertices=4_000_000, degree=8, skew=False, sources=40_000,
             max_hops=NEVER),
        # Interaction-involved simulation: agents on a tile grid, uniform, and a
        # larger population gathered around places.
        dict(name="interaction_50k", kind="interaction", agents=50_000, side=2048, places=0,
             velocity=3, radius=2),
        dict(name="interaction_200k", kind="interaction", agents=200_000, side=8192, places=400,
             velocity=2, radius=4),
    ]


def _between(rng, lo, hi):
    """A whole number spread over the logarithm of [lo, hi]."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _due(agents, active, period):
    """Agents that become active in a period, on average."""
    return agents * (1 - (1 - active / agents) ** period)


def draw(rng):
    kind = rng.choice(["step", "step", "step", "loader", "objects", "hops", "interaction"])
    if kind == "step":
        agents = _between(rng, 40, 60_000)
        hi = rng.randint(1, max(1, min(40, 150_000 // agents)))
        lo = rng.randint(1, hi)
        mean = (lo + hi) / 2
        # pages from one 16 KiB plane to a large model's 2 MiB, as far as the
        # host copies of all agents stay within 1.5 GB
        pages = [(1, 16 * KIB), (4, 4 * KIB), (3, 1040), (6, 8 * KIB), (1, 512 * KIB),
                 (16, 32 * KIB), (5, 48 * KIB), (64, 32 * KIB)]
        pages = [p for p in pages if p[0] * p[1] * mean * agents < 1.5e9] or pages[2:3]
        planes, chunk = rng.choice(pages)
        active = max(1, min(int(agents * rng.uniform(0.002, 0.1)), 1000))
        period = rng.randint(12, 48)
        # a pool of less than what becomes active in a period
        capacity = max(4 * hi, int(_due(agents, active, period) * mean * rng.uniform(0.2, 0.8)),
                       int(2 * active * mean))
        budget = rng.choice([0, 0, rng.randint(1, 200)])
        steps = period if active * mean * planes * chunk > 4 * MIB else 1
        return dict(kind="step", agents=agents, units_lo=lo, units_hi=hi, planes=planes,
                    chunk=chunk, capacity=capacity, active=active, period=period, steps=steps,
                    noise=rng.choice([0, 2]),
                    threshold=rng.choice([0, rng.randint(1, 12), NEVER]) if budget == 0
                    else rng.choice([rng.randint(2, 12), NEVER]),
                    budget=budget, inputs=rng.choice(["device", "host"]),
                    dirty=rng.choice(["all", "half"]), shared=0,
                    direct=rng.choice([0, 4 * MIB, 4 * MIB]),
                    slot_units=max(8, min(1024, (64 * MIB) // (planes * chunk))),
                    ring=rng.randint(2, 4))
    if kind == "loader":
        planes, chunk = rng.choice([(64, 32 * KIB), (16, 32 * KIB), (1, 512 * KIB), (4, 4 * KIB)])
        agents = rng.randint(8, 40)
        hi = rng.randint(4, 32)
        return dict(kind="loader", agents=agents, units_lo=rng.randint(1, hi), units_hi=hi,
                    planes=planes, chunk=chunk, urgent=rng.randint(1, 6),
                    slot_units=rng.randint(2, 32), ring=rng.randint(2, 4))
    if kind == "objects":
        return dict(kind="objects", trees=_between(rng, 1, 40), agents=_between(rng, 300, 50_000),
                    branching=rng.randint(2, 12), depth=rng.randint(2, 6),
                    active=round(rng.uniform(0.002, 0.1), 4))
    if kind == "hops":
        vertices = _between(rng, 500, 3_000_000)
        return dict(kind="hops", vertices=vertices, degree=rng.randint(2, 12),
                    skew=rng.random() < 0.5,
                    sources=max(1, int(vertices * rng.choice([0.0, 0.001, 0.01, 0.05]))),
                    max_hops=rng.choice([NEVER, NEVER, rng.randint(1, 6)]))
    agents = _between(rng, 200, 200_000)
    return dict(kind="interaction", agents=agents, side=_between(rng, 100, 32_768),
                places=rng.choice([0, _between(rng, 1, 500)]), velocity=rng.randint(1, 6),
                radius=rng.randint(0, 8))


_stream = None


def _caller_stream():
    """The one stream that the program queues everything on."""
    global _stream
    if _stream is None:
        _stream = torch.cuda.Stream()
    return _stream.cuda_stream


class _Memory:
    """The memory of a pool or loader and the pool or loader itself, which is
    closed before its memory goes."""

    owner = None

    def __del__(self):
        if self.owner is not None:
            self.owner.close()


class _View:
    """A pool's device memory as an array for torch, which keeps the pool."""

    def __init__(self, ptr, shape, kind, memory):
        self.memory = memory
        self.__cuda_array_interface__ = dict(data=(ptr, False), shape=shape, typestr=kind,
                                             version=2)


class _State:
    """What a program keeps between calls."""

    def __init__(self, case):
        self.case = case


def _fill_host(words, rng):
    """Pseudo-random bytes over all host copies; the pattern's length is odd
    in every page size, so no two pages are alike."""
    pattern = rng.integers(-(1 << 62), 1 << 62, size=(8 << 20) // 8 + 513)
    for at in range(0, len(words), len(pattern)):
        n = min(len(pattern), len(words) - at)
        words[at:at + n] = pattern[:n]


def _memory(case, rng, units, capacity, host_copies):
    """Planes, staging and host copies, and the arguments that describe them."""
    mem = _Memory()
    chunk, planes = case["chunk"], case["planes"]
    unit_bytes = chunk * planes
    plane = (capacity * chunk + 255) // 256 * 256
    mem.arena = torch.zeros(planes * plane // 8, dtype=torch.int64, device="cuda")
    slot = case["slot_units"] * unit_bytes
    mem.staging = torch.zeros((2 * case["ring"] * slot + 256) // 8, dtype=torch.int64,
                              device="cuda")
    size = units.astype(np.uint64) * np.uint64(unit_bytes)
    if host_copies:
        off = (np.arange(len(units), dtype=np.uint64) % np.uint64(host_copies)) * size.max()
        host_bytes = int(host_copies * size.max())
    else:
        off = np.concatenate([[0], np.cumsum(size)[:-1]]).astype(np.uint64)
        host_bytes = int(size.sum())
    mem.host = torch.empty(host_bytes // 8, dtype=torch.int64, pin_memory=True)
    _fill_host(mem.host.numpy(), rng)
    return mem, dict(capacity_units=capacity, chunk_bytes=[chunk] * planes, agent_units=units,
                     plane_base=[mem.arena.data_ptr() + c * plane for c in range(planes)],
                     host_backing=mem.host.data_ptr(), host_bytes=host_bytes, host_off=off,
                     dev_staging=mem.staging.data_ptr(), staging_bytes=2 * case["ring"] * slot,
                     ring_slots=case["ring"])


def _sizes(case, rng):
    """Agents' units, spread evenly over their range, in random order."""
    n, lo, hi = case["agents"], case["units_lo"], case["units_hi"]
    return rng.permutation(lo + np.arange(n) * (hi - lo + 1) // n).astype(np.uint32)


def _prepare_step(case, seed):
    s = _State(case)
    rng = np.random.default_rng(seed)
    n, steps = case["agents"], case["period"]
    units = _sizes(case, rng)
    s.mem, desc = _memory(case, rng, units, case["capacity"], case["shared"])
    torch.cuda.synchronize()
    s.mem.owner = s.pool = binding.Pool(**desc, direct_bytes=case["direct"])
    active = np.zeros((steps, n), dtype=np.uint8)
    for t in range(steps):
        # half of a step's agents are a burst of neighbours, half anywhere
        who = np.concatenate([(rng.integers(n) + np.arange(case["active"] // 2)) % n,
                              rng.choice(n, case["active"] - case["active"] // 2, replace=False)])
        who = who[np.cumsum(units[who].astype(np.int64)) <= case["capacity"] * 3 // 4]
        active[t, who] = 1
    # the schedule repeats: steps to the next activation; agents that are not
    # due in it are due some time later, a tenth of them never
    far = steps + rng.geometric(0.02, size=n) + steps
    far[rng.random(n) < 0.1] = NEVER
    dist = np.empty((steps, n), dtype=np.int64)
    due = active.any(0)
    nxt = np.where(due, active.argmax(0) + steps, 0)
    for t in range(steps - 1, -1, -1):
        dist[t] = np.where(due, nxt - t, np.where(far == NEVER, NEVER, far - t))
        nxt = np.where(active[t] != 0, t, nxt)
    if case["noise"]:
        noisy = np.maximum(1, dist + np.rint(rng.normal(0, case["noise"], dist.shape)).astype(int))
        dist = np.where(dist == NEVER, NEVER, noisy)
    dist = dist.astype(np.uint32)
    dirty = None if case["dirty"] == "all" else (
        rng.random(n) < (0.5 if case["dirty"] == "half" else 0.0)).astype(np.uint8)
    s.keep = (dist, active, dirty)
    if case["inputs"] == "device":
        s.keep = tuple(None if x is None else torch.from_numpy(x.view(np.uint8)).cuda()
                       for x in s.keep)
        at = [0 if x is None else x.data_ptr() for x in s.keep]
    else:
        at = [0 if x is None else x.ctypes.data for x in s.keep]
    s.at = [(at[0] + 4 * n * t, at[1] + n * t) for t in range(steps)]
    s.dirty = at[2]
    bt, _ = s.pool.block_table()
    s.table = torch.as_tensor(_View(bt, (int(units.sum()),), "<i4", s.mem), device="cuda")
    s.lists = [np.zeros(n, dtype=np.int32) for _ in range(3)]
    s.t = 0
    torch.cuda.synchronize()
    for _ in range(steps):          # the pool is full from here on
        _one_step(s)
    s.pool.sync()
    return s


def _run_step(s):
    for _ in range(s.case["steps"]):
        counts = _one_step(s)
    return {"counts": counts, "lists": s.lists, "table": s.table, "pool": s.mem.arena,
            "host": s.mem.host}


def _one_step(s):
    c, pool, st = s.case, s.pool, _caller_stream()
    dist, active = s.at[s.t % len(s.at)]
    s.t += 1
    plan = pool.plan_step(dist, active, c["threshold"], c["budget"] or None, st, s.dirty)
    pool.evict_pack(st)
    pool.prefetch_unpack(st)
    # the plan's lists, at the front of arrays that hold any plan
    for to, name in zip(s.lists, ("victims", "loads", "victim_written")):
        to[:len(plan[name])] = plan[name]
        to[len(plan[name]):] = -1
    return [plan[k] for k in ("n_victims", "n_loads", "n_demand", "n_demand_victims", "units_out",
                              "units_in", "units_written", "bytes_out", "bytes_in")]


def _prepare_loader(case, seed):
    s = _State(case)
    rng = np.random.default_rng(seed)
    n = case["agents"]
    units = _sizes(case, rng)
    total = int(units.sum())
    s.mem, desc = _memory(case, rng, units, total, 0)
    torch.cuda.synchronize()
    s.mem.owner = s.loader = binding.Loader([desc])
    s.units = torch.from_numpy(rng.permutation(total).astype(np.int32)).cuda()
    at = s.units.data_ptr() + 4 * np.concatenate([[0], np.cumsum(units)[:-1]]).astype(np.int64)
    dist = rng.integers(1, 50, size=n)
    who = rng.permutation(n)
    s.background = [(0, int(a), int(dist[a]), int(at[a])) for a in who[case["urgent"]:]]
    s.urgent = [(0, int(a), 0, int(at[a])) for a in who[:case["urgent"]]]
    s.chunks = int(((units + case["slot_units"] - 1) // case["slot_units"]).sum()) + n
    torch.cuda.synchronize()
    return s


def _run_loader(s):
    L = s.loader
    L.submit(s.background)
    log = L.pump(3)
    L.submit(s.urgent)
    log += L.pump(s.chunks)
    return {"log": np.array(log, dtype=np.int64), "pool": s.mem.arena}


def _prepare_objects(case, seed):
    s = _State(case)
    rng = np.random.default_rng(seed)
    n, trees = case["agents"], case["trees"]
    paths = rng.integers(0, case["branching"], size=(n, case["depth"]))
    code, lists, ends, total = np.zeros(n, dtype=np.int64), [], [], 0
    for level in range(case["depth"] + 1):      # a tree's nodes by depth, then by path
        if level:
            code = code * case["branching"] + paths[:, level - 1]
        order = np.argsort(code, kind="stable")
        lists.append(order)
        ends.append(total + np.cumsum(np.unique(code, return_counts=True)[1]))
        total += n
    lists.append(np.arange(n))                   # one private leaf per agent
    ends.append(total + np.arange(1, n + 1))
    ends = torch.from_numpy(np.concatenate(ends)).cuda()
    refs = torch.from_numpy(np.concatenate(lists)).cuda()
    k = torch.arange(trees, device="cuda").view(-1, 1)
    off = torch.cat([torch.zeros(1, dtype=torch.int64, device="cuda"),
                     (ends + k * len(refs)).view(-1)])
    s.off = off.to(torch.int32)
    s.refs = (refs + k * n).view(-1).to(torch.int32)
    s.n = n * trees
    g = torch.Generator(device="cuda").manual_seed(seed)
    s.dist = torch.randint(1, 1 << 20, (s.n,), generator=g, device="cuda", dtype=torch.int32)
    s.active = (torch.rand(s.n, generator=g, device="cuda") < case["active"]).to(torch.uint8)
    s.m = m = len(s.off) - 1
    # room for the objects of any such forest
    most = trees * (sum(min(n, case["branching"] ** k) for k in range(case["depth"] + 1)) + n)
    s.out = torch.zeros(most, dtype=torch.int32, device="cuda")
    s.out_active = torch.zeros(most, dtype=torch.uint8, device="cuda")
    s.ws = torch.empty(binding.object_distances_workspace(m, len(s.refs), s.n), dtype=torch.uint8,
                       device="cuda")
    return s


def _run_objects(s):
    binding.object_distances(s.off.data_ptr(), s.refs.data_ptr(), s.m, len(s.refs),
                             s.dist.data_ptr(), s.active.data_ptr(), s.n, s.out.data_ptr(),
                             s.out_active.data_ptr(), s.ws.data_ptr(), len(s.ws),
                             _caller_stream())
    return {"distances": s.out, "active": s.out_active}


def _prepare_hops(case, seed):
    s = _State(case)
    g = torch.Generator(device="cuda").manual_seed(seed)
    v, d = case["vertices"], case["degree"]
    if case["skew"]:                             # most agents message few, some message many
        u = torch.rand(v, generator=g, device="cuda")
        deg = (d * 0.4 / (u + 0.02).sqrt()).floor().to(torch.int64)
    else:
        deg = torch.full((v,), d, dtype=torch.int64, device="cuda")
    off = torch.zeros(v + 1, dtype=torch.int64, device="cuda")
    off[1:] = deg.cumsum(0)
    e = int(off[-1])
    s.off = off.to(torch.int32)
    s.col = torch.randint(0, v, (e,), generator=g, device="cuda", dtype=torch.int32)
    s.src = torch.randperm(v, generator=g, device="cuda")[:case["sources"]].to(torch.int32)
    s.hops = torch.zeros(v, dtype=torch.int32, device="cuda")
    s.ws = torch.empty(binding.hop_distances_workspace(v), dtype=torch.uint8, device="cuda")
    return s


def _run_hops(s):
    binding.hop_distances(s.off.data_ptr(), s.col.data_ptr(), len(s.hops), len(s.col),
                          s.src.data_ptr(), len(s.src), s.case["max_hops"], s.hops.data_ptr(),
                          s.ws.data_ptr(), len(s.ws), _caller_stream())
    return s.hops


def _prepare_interaction(case, seed):
    s = _State(case)
    g = torch.Generator(device="cuda").manual_seed(seed)
    n, side = case["agents"], case["side"]
    pos = torch.rand(n, 2, generator=g, device="cuda") * side
    if case["places"]:                           # three in four agents near a place
        place = torch.rand(case["places"], 2, generator=g, device="cuda") * side
        at = torch.randint(0, case["places"], (n,), generator=g, device="cuda")
        near = place[at] + torch.randn(n, 2, generator=g, device="cuda") * (side / 200)
        pos = torch.where(torch.rand(n, 1, generator=g, device="cuda") < 0.75, near, pos)
    s.pos = pos.to(torch.int32).clamp_(0, side - 1).contiguous()
    s.action = torch.randint(0, 1000, (n,), generator=g, device="cuda", dtype=torch.int32)
    s.out = torch.zeros(n, dtype=torch.int32, device="cuda")
    s.ws = torch.empty(binding.interaction_distances_workspace(n), dtype=torch.uint8,
                       device="cuda")
    return s


def _run_interaction(s):
    c = s.case
    binding.interaction_distances(s.pos.data_ptr(), s.action.data_ptr(), c["agents"],
                                  c["velocity"], c["radius"], s.out.data_ptr(), s.ws.data_ptr(),
                                  len(s.ws), _caller_stream())
    return s.out


def prepare(case, seed):
    return globals()["_prepare_" + case["kind"]](case, seed)


def run(state):
    return globals()["_run_" + state.case["kind"]](state)


def work(case):
    """Bytes that a pass reads and writes once.  Of a step: its inputs, and
    the memory of the agents that become active and are not in the pool (on
    average: what becomes active in a period and does not fit), over the host
    link and in the pool, both ways when what they replace is written back.
    Plain integer work throughout: no products."""
    n = case.get("agents", 0)
    if case["kind"] == "step":
        mean = (case["units_lo"] + case["units_hi"]) / 2
        due = _due(n, case["active"], case["period"]) * mean
        moved = max(0.0, due - case["capacity"]) / case["period"] * case["planes"] * case["chunk"]
        ways = {"all": 2, "half": 1.5, "none": 1}[case["dirty"]]
        return {"bytes": case["steps"] * (10 * n + 2 * ways * moved), "flops": 0}
    if case["kind"] == "loader":
        mean = (case["units_lo"] + case["units_hi"]) / 2
        return {"bytes": 2 * n * mean * case["planes"] * case["chunk"], "flops": 0}
    if case["kind"] == "objects":
        b, d = case["branching"], case["depth"]
        # nodes that some agent's path meets, and the private leaves
        nodes = sum(b ** k * (1 - (1 - b ** -k) ** n) if k else 1 for k in range(d + 1)) + n
        refs = n * (d + 2)
        return {"bytes": case["trees"] * (9 * nodes + 4 * refs + 5 * n), "flops": 0}
    if case["kind"] == "hops":
        return {"bytes": case["vertices"] * (8 + 4 * case["degree"]) + 4 * case["sources"],
                "flops": 0}
    return {"bytes": 16 * n, "flops": 0}


def tolerance(case):
    return "exact"


def exact(case, seed):
    return None                  # whole numbers and moved bytes: compared as they are
