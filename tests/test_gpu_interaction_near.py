"""The two paths of ss_interaction_distances, all pairs and the search by
cells, against a k-d tree's nearest neighbours (exact in integers), at the sizes
and distributions where either can go wrong."""
import numpy as np
import pytest

from paper_2601_21473_amd import binding as B
from paper_2601_21473_amd.memory import DeviceBuffer

pytestmark = pytest.mark.gpu
NEVER = 0xFFFFFFFF
NEAR = 32768                        # agents from which the search by cells runs


def places(kind, n, rng):
    if kind == "even":
        return rng.integers(0, 2048, (n, 2))
    if kind == "wide":              # about one agent per block of 512 x 512 tiles and more
        return rng.integers(0, 32768, (n, 2))
    if kind == "one tile":
        return np.full((n, 2), 32767)
    if kind == "column":
        return np.stack([np.full(n, 511), rng.integers(0, 32768, n)], 1)
    if kind == "lattice":           # every nearest agent two tiles off, over block edges
        side = int(np.ceil(n ** 0.5))
        i = np.arange(n)
        return np.stack([i % side, i // side], 1) * 2 + 300
    if kind == "crowd":             # a crowd on a few tiles, lone agents beside it
        p = rng.integers(1000, 1004, (n, 2))
        p[:200] = rng.integers(990, 1020, (200, 2))
        return p
    assert kind == "town"           # dense, and a few agents anywhere
    p = rng.integers(400, 400 + max(2, int(n ** 0.5)), (n, 2))
    p[:6] = [[0, 0], [32767, 32767], [32767, 450], [450, 20000], [390, 390], [12000, 13000]]
    return p


def expected(pos, d_act, velocity, radius):
    from scipy.spatial import cKDTree
    d = cKDTree(pos).query(pos, k=2)[0][:, 1]
    d2 = np.rint(d * d).astype(np.int64)
    root = np.floor(np.sqrt(d2.astype(np.float64))).astype(np.int64)
    root -= root * root > d2
    root += (root + 1) * (root + 1) <= d2
    return np.minimum(d_act.astype(np.int64), np.maximum(0, root - radius) // velocity)


@pytest.mark.parametrize("n,kind", [
    (2, "wide"), (15, "even"), (17, "even"), (65, "wide"), (12288, "even"), (12289, "even"),
    (NEAR - 1, "town"), (NEAR, "even"), (NEAR, "wide"), (NEAR, "one tile"), (NEAR, "lattice"),
    (NEAR + 1, "town"), (NEAR + 1, "crowd"), (NEAR + 1, "column"), (36865, "wide"),
    (131072, "even"), (131073, "town"), (131073, "wide")])
def test_nearest_agent(n, kind):
    rng = np.random.default_rng(n)
    pos = np.ascontiguousarray(places(kind, n, rng), dtype=np.int32)
    d_act = rng.integers(0, 1 << 16, n).astype(np.uint32)
    d_act[::3] = NEVER
    exp = expected(pos, d_act, 1, 0)
    p, d, out = DeviceBuffer(8 * n), DeviceBuffer(4 * n), DeviceBuffer(4 * n)
    full = B.interaction_distances_workspace(n)
    ws = DeviceBuffer(full)
    try:
        p.upload(pos.reshape(-1))
        ws.upload(np.full(full, 0x77, np.uint8))
        for label, call in [
                ("workspace", lambda o: B.interaction_distances(p.ptr, d.ptr, n, 1, 0, o, ws.ptr,
                                                                full)),
                ("again", lambda o: B.interaction_distances(p.ptr, d.ptr, n, 1, 0, o, ws.ptr, full)),
                ("all pairs", lambda o: B.interaction_distances(p.ptr, d.ptr, n, 1, 0, o, ws.ptr,
                                                                4 * n)),
                ("static", lambda o: B.interaction_distances_static(p.ptr, d.ptr, n, 1, 0, o)),
                ("in place", lambda o: B.interaction_distances(p.ptr, d.ptr, n, 1, 0, d.ptr, ws.ptr,
                                                               full))]:
            print(f"[interaction] n={n} {kind} {label}", flush=True)
            d.upload(d_act)
            call(out.ptr)
            got = (d if label == "in place" else out).download(0, 4 * n).view(np.uint32)
            bad = np.flatnonzero(got != exp)
            assert len(bad) == 0, (label, bad[:5], pos[bad[:5]], got[bad[:5]], exp[bad[:5]])
    finally:
        for b in (p, d, out, ws):
            b.free()


@pytest.mark.parametrize("n", [1, 700, NEAR + 5])
def test_positions_at_any_word(n):
    """Positions on a 4-byte boundary that is no 8-byte one: both paths."""
    rng = np.random.default_rng(n)
    pos = np.ascontiguousarray(places("even", n, rng), dtype=np.int32)
    d_act = np.full(n, 60, np.uint32)
    exp = expected(pos, d_act, 1, 0) if n > 1 else d_act
    p, d, out = DeviceBuffer(8 * n + 4), DeviceBuffer(4 * n), DeviceBuffer(4 * n)
    full = B.interaction_distances_workspace(n)
    ws = DeviceBuffer(full)
    try:
        p.upload(pos.reshape(-1), 4)
        d.upload(d_act)
        for size in (4 * n, full):
            B.interaction_distances(p.ptr + 4, d.ptr, n, 1, 0, out.ptr, ws.ptr, size)
            assert np.array_equal(out.download(0, 4 * n).view(np.uint32), exp)
    finally:
        for b in (p, d, out, ws):
            b.free()


def test_short_workspace_is_refused():
    n = NEAR
    b = DeviceBuffer(16 * n)
    try:
        with pytest.raises(B.ScaleSimError) as e:
            B.interaction_distances(b.ptr, b.ptr, n, 1, 0, b.ptr, b.ptr, 4 * n - 1)
        assert e.value.status == B.SS_ERR_ARG
    finally:
        b.free()
