"""The agents' 32-bit words of ss_object_distances: the two largest distances,
which share a word, and arrays that the four-agent reads cannot take, at agent
counts around a workgroup's 2,048."""
import numpy as np
import pytest

from oracle.objects import object_distances
from paper_2601_21473_amd import binding as B
from paper_2601_21473_amd.memory import DeviceBuffer

pytestmark = pytest.mark.gpu
S = 0xFFFFFFFF


@pytest.mark.parametrize("n", [1, 2047, 2048, 2049, 6145])
@pytest.mark.parametrize("shift", [0, 1])       # agents that dist and active start late by
@pytest.mark.parametrize("odd", [0, 1, 400])    # agents at the second largest distance
def test_words(n, shift, odd):
    rng = np.random.default_rng(n + odd)
    dist = rng.choice(np.array([0, 1, 7, S - 2, S], np.uint32), n)
    act = (rng.random(n) < 0.1).astype(np.uint8)
    who = rng.choice(n, min(odd, n), replace=False)
    dist[who] = S - 1
    act[who[::2]] = 0
    # every agent alone, pairs, one large group of those far away, an empty row
    far = np.flatnonzero((dist >= S - 1) & (act == 0))
    lists = [[a] for a in range(n)] + [rng.integers(0, n, 2).tolist() for _ in range(300)]
    lists += [far.tolist(), [], rng.integers(0, n + 3, 50).tolist()]
    off = np.concatenate([[0], np.cumsum([len(x) for x in lists])]).astype(np.uint32)
    agents = np.concatenate([np.asarray(x, np.uint32) for x in lists])
    m = len(lists)
    bufs = [DeviceBuffer(a.nbytes) for a in (off, agents)]
    d_dist, d_act = DeviceBuffer(4 * (n + shift)), DeviceBuffer(n + shift)
    d_out, d_oa = DeviceBuffer(4 * m), DeviceBuffer(m)
    wsb = B.object_distances_workspace(m, len(agents), n)
    ws = DeviceBuffer(wsb)
    try:
        bufs[0].upload(off)
        bufs[1].upload(agents)
        d_dist.upload(dist, 4 * shift)
        d_act.upload(act, shift)
        ws.upload(np.full(wsb, 0x77, np.uint8))
        for _ in range(2):
            B.object_distances(bufs[0].ptr, bufs[1].ptr, m, len(agents), d_dist.ptr + 4 * shift,
                               d_act.ptr + shift, n, d_out.ptr, d_oa.ptr, ws.ptr, wsb)
            exp_d, exp_a = object_distances(off, agents, dist, act)
            assert np.array_equal(d_out.download(0, 4 * m).view(np.uint32), exp_d)
            assert np.array_equal(d_oa.download(0, m), exp_a)
    finally:
        for b in bufs + [d_dist, d_act, d_out, d_oa, ws]:
            b.free()


@pytest.mark.parametrize("n", [2, 3, 4, 5, 2046, 2050, 300_003, 1_060_001])
def test_last_agents(n):
    """The one to three agents that no four-agent read takes, and the flags of many
    preparing workgroups (518 in the last case): only the last agent, or the last
    of a wave, has the second largest distance."""
    rng = np.random.default_rng(n)
    base = rng.choice(np.array([5, S - 2, S], np.uint32), n)
    act = np.zeros(n, np.uint8)
    act[rng.integers(0, n, n // 10)] = 1
    some = np.unique(np.concatenate([np.arange(max(0, n - 6), n), rng.integers(0, n, 500)]))
    never = np.flatnonzero(base == S)[:3000]
    lists = [[a] for a in some] + [never.tolist(), never[-4:].tolist() + [n - 1], []]
    off = np.concatenate([[0], np.cumsum([len(x) for x in lists])]).astype(np.uint32)
    agents = np.concatenate([np.asarray(x, np.uint32) for x in lists])
    m = len(lists)
    bufs = [DeviceBuffer(b) for b in (off.nbytes, agents.nbytes, 4 * n, n, 4 * m, m)]
    wsb = B.object_distances_workspace(m, len(agents), n)
    ws = DeviceBuffer(wsb)
    try:
        bufs[0].upload(off)
        bufs[1].upload(agents)
        for at in (None, n - 1, min(n - 1, 63 * 4 + 3)):
            dist = base.copy()
            if at is not None:
                dist[at] = S - 1
                act[at] = 0
            bufs[2].upload(dist)
            bufs[3].upload(act)
            ws.upload(np.full(wsb, 0x77, np.uint8))
            B.object_distances(bufs[0].ptr, bufs[1].ptr, m, len(agents), bufs[2].ptr, bufs[3].ptr, n,
                               bufs[4].ptr, bufs[5].ptr, ws.ptr, wsb)
            exp_d, exp_a = object_distances(off, agents, dist, act)
            assert np.array_equal(bufs[4].download(0, 4 * m).view(np.uint32), exp_d), at
            assert np.array_equal(bufs[5].download(0, m), exp_a), at
    finally:
        for b in bufs + [ws]:
            b.free()
