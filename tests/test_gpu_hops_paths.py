"""ss_hop_distances at the sizes where its paths change: the edges of the
stretches of vertices, the first sizes with the visited hint and with larger
stretches, and the frontier queues of very large graphs."""
import numpy as np
import pytest

from oracle.estimators import hop_distances
from paper_2601_21473_amd import binding as B
from paper_2601_21473_amd.memory import DeviceBuffer

pytestmark = pytest.mark.gpu
NEVER = 0xFFFFFFFF


def gpu_hops(off, col, src, max_hops=NEVER, calls=2, probe=None):
    """``probe``: (workgroups, polls) of ``probe_hop_distances``."""
    v, e = len(off) - 1, len(col)
    bufs = [DeviceBuffer(4 * (v + 1)), DeviceBuffer(max(4, 4 * e)), DeviceBuffer(max(4, 4 * len(src))),
            DeviceBuffer(4 * v)]
    wsb = B.hop_distances_workspace(v)
    ws = DeviceBuffer(wsb)
    try:
        for b, a in zip(bufs, (off, col, src)):
            if len(a):
                b.upload(np.asarray(a, np.uint32))
        ws.upload(np.full(min(wsb, 1 << 20), 0x77, np.uint8))
        out = []
        for _ in range(calls):                  # the second call finds the first one's workspace
            args = (bufs[0].ptr, bufs[1].ptr, v, e, bufs[2].ptr, len(src), max_hops, bufs[3].ptr,
                    ws.ptr, wsb)
            if probe:
                B.probe_hop_distances(*args, *probe)
            else:
                B.hop_distances(*args)
            out.append(bufs[3].download(0, 4 * v).view(np.uint32))
            assert ws.download(20, 4).view(np.uint32)[0] == 0
        for h in out[1:]:
            assert np.array_equal(h, out[0])
        return out[0]
    finally:
        for b in bufs + [ws]:
            b.free()


@pytest.mark.parametrize("v", [1, 2, 1023, 1024, 1025, 2049, 32_767, 32_768, 98_304, 98_305])
@pytest.mark.parametrize("shape", ["random", "hub", "ring"])
def test_stretches(v, shape):
    rng = np.random.default_rng(v)
    if shape == "random":
        deg = rng.integers(0, 12, v)
    elif shape == "hub":                        # one vertex with thousands of edges, few others
        deg = (rng.random(v) < 0.5).astype(np.int64)
        deg[v // 2] = min(5000, 3 * v)
    else:
        deg = np.ones(v, np.int64)
    off = np.concatenate([[0], np.cumsum(deg)])
    col = rng.integers(0, v, off[-1]).astype(np.uint32)
    src = rng.integers(0, v + 2, max(1, v // 200))       # repeated and foreign ids too
    if shape == "hub":
        src[0] = v // 2
    if shape == "ring":
        step = max(1, v // 60)
        col = ((np.arange(v) + step) % v).astype(np.uint32)
        src = np.arange(step)
    for max_hops in (None, 0, 3):
        print(f"[hops] v={v} {shape} max_hops={max_hops}", flush=True)
        got = gpu_hops(off, col, src, NEVER if max_hops is None else max_hops)
        exp = hop_distances(off, col, src, max_hops)
        bad = np.flatnonzero(got != exp)
        assert len(bad) == 0, (bad[:5], got[bad[:5]], exp[bad[:5]])


@pytest.mark.parametrize("v", [(1 << 22), (1 << 22) + 1])
def test_very_large_ring(v):
    """Closed form: on a ring of step w from its first w vertices, vertex i is
    i // w hops away."""
    w = 120_000
    got = gpu_hops(np.arange(v + 1), (np.arange(v) + w) % v, np.arange(w), calls=1)
    assert np.array_equal(got, np.arange(v) // w)


@pytest.mark.parametrize("v", [2048, 5000, 40_000])
def test_wait_bound_grows_with_the_graph(v):
    """A vertex of a million edges keeps its workgroup longer than any wait
    bound without regard to the graph would allow here (0 polls): the others
    wait for it all the same."""
    rng = np.random.default_rng(v)
    deg = np.full(v, 2)
    deg[v // 2] = 1_000_000
    off = np.concatenate([[0], np.cumsum(deg)])
    col = rng.integers(0, v, off[-1])
    print(f"[hops] v={v} hub, 0 polls", flush=True)
    got = gpu_hops(off, col, [v // 2], calls=1, probe=(512, 0))
    assert np.array_equal(got, hop_distances(off, col, np.array([v // 2]), None))


def communities(v, size, degree, seed):
    """Edges inside blocks of ``size`` consecutive vertices, and from every 64th
    vertex one into the next block."""
    rng = np.random.default_rng(seed)
    col = (np.arange(v) // size * size)[:, None] + rng.integers(0, size, (v, degree))
    col[::64, 0] = np.arange(0, v, 64) + size
    return np.arange(v + 1) * degree, np.minimum(col, v - 1)


@pytest.mark.parametrize("v,size", [(30_000, 500), (300_000, 4096), (300_000, 70_000)])
def test_communities(v, size):
    """Levels that lie close together in the vertices' numbers."""
    off, col = communities(v, size, 6, v)
    col = col.reshape(-1)
    for src in ([0], [v // 2, 5]):
        got = gpu_hops(off, col, src)
        assert np.array_equal(got, hop_distances(off, col, np.array(src), None))


def test_time_does_not_depend_on_the_numbering():
    """A search whose levels lie close together takes at most twice as long as
    over the same graph with its vertices numbered at random (it took four times
    as long where every level was the work of one or two workgroups)."""
    v, degree = 1 << 22, 8
    off, col = communities(v, 16384, degree, 1)
    to = np.random.default_rng(2).permutation(v)
    mixed = np.empty_like(col)
    mixed[to] = to[col]
    ms, hops = [], []
    timer = B.EventTimer()
    for c, s in ((col, 0), (mixed, to[0])):
        bufs = [DeviceBuffer(4 * (v + 1)), DeviceBuffer(4 * v * degree), DeviceBuffer(4),
                DeviceBuffer(4 * v)]
        wsb = B.hop_distances_workspace(v)
        ws = DeviceBuffer(wsb)
        try:
            for b, a in zip(bufs, (off, c.reshape(-1), [s])):
                b.upload(np.asarray(a, np.uint32))
            times = []
            for _ in range(4):
                with timer:
                    B.hop_distances(bufs[0].ptr, bufs[1].ptr, v, v * degree, bufs[2].ptr, 1, NEVER,
                                    bufs[3].ptr, ws.ptr, wsb, timer.handle)
                times.append(timer.ms)
            ms.append(min(times[1:]))
            hops.append(bufs[3].download(0, 4 * v).view(np.uint32))
        finally:
            for b in bufs + [ws]:
                b.free()
    timer.close()
    print(f"[hops] by community {ms[0]:.2f} ms, at random {ms[1]:.2f} ms", flush=True)
    assert np.array_equal(hops[0], hops[1][to])
    assert ms[0] <= 2 * ms[1], ms


@pytest.mark.parametrize("v,workgroups", [(2048, 1), (5000, 2), (40_000, 1), (40_000, 7),
                                          (300_000, 1), (300_000, 50)])
def test_fewer_workgroups_than_chunks(v, workgroups):
    """As when the device is busy: the workgroups that run draw the tickets of
    those that never do."""
    rng = np.random.default_rng(v)
    deg = rng.integers(0, 8, v)
    off = np.concatenate([[0], np.cumsum(deg)])
    col = rng.integers(0, v, off[-1])
    src = rng.integers(0, v, 5)
    got = gpu_hops(off, col, src, probe=(workgroups, 1 << 22))
    assert np.array_equal(got, hop_distances(off, col, src, None))


@pytest.mark.parametrize("v,degree", [(70, 8000), (1000, 1000), (2100, 300)])
def test_dense_graphs(v, degree):
    """Chunks of fewer than 1,024 vertices, down to one stretch of 64."""
    rng = np.random.default_rng(v)
    off = np.arange(v + 1) * degree
    # most edges stay near, so that the search takes some levels
    col = (np.arange(v)[:, None] + rng.integers(0, 9, (v, degree))) % v
    col[:, 0] = rng.integers(0, v, v)
    got = gpu_hops(off, col.reshape(-1), [v // 3])
    assert np.array_equal(got, hop_distances(off, col.reshape(-1), np.array([v // 3]), None))
