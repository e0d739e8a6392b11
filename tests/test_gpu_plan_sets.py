"""Plan kernels at the edges of their agent counts and sorted sets, against the
oracle's plans and bytes."""
import numpy as np
import pytest

import workloads as W
from gpu_harness import S, run_parity

pytestmark = pytest.mark.gpu


def ragged_trace(n, per_step, seed, steps=14):
    """per_step random agents of 1 to 4 units a step (none at step 5), a pool of
    a third more than the largest step needs."""
    rng = np.random.default_rng(seed)
    units = rng.integers(1, 5, n).astype(np.uint32)
    active = np.zeros((steps, n), np.uint8)
    for t in range(steps):
        if t != 5:
            active[t, rng.choice(n, per_step, replace=False)] = 1
    need = int((active.astype(np.int64) * units).sum(1).max())
    pool = W.PoolSpec("syn", need + need // 3 + 1, [16], units)
    dist = W.exact_distances(active)
    return W.Trace(f"sets{n}", n, steps, [pool], active, dist, dist.copy(), {})


# around a wave, the sort's register runs and one agent per thread of the
# workgroup (1,024: the plan that sorts every agent; above it the cuts)
@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 129, 512, 513, 1023, 1024, 1025])
@pytest.mark.parametrize("theta,budget,dirty", [
    (S, None, False), (6, 17, True), (0, None, False), (S, 0, True)])
def test_small_plans(n, theta, budget, dirty):
    tr = ragged_trace(n, max(1, n // 3), n)
    mask = None
    if dirty:                                   # some steps' victims partly written back
        mask = (np.random.default_rng(n + 1).random((tr.n_steps, n)) < 0.5).astype(np.uint8)
    run_parity(tr, theta=theta, budget=budget, slot_units=64, ring_slots=2, dirty=mask,
               check_mirrors=True, label=f"small plan {n}, threshold {theta}, budget {budget}")


# The union of the sets that a plan of n unit-size agents sorts is n keys here
# (see the sets of test_joint_sort_sizes): the last union in LDS is 8,191 keys.
@pytest.mark.parametrize("n", [8190, 8191, 8192, 8193])
def test_joint_sort_edge(n):
    cap = 4100
    active = np.zeros((4, n), np.uint8)
    active[0, :cap] = 1
    active[1, cap:cap + 100] = 1
    active[2, cap + 100:] = 1
    dist = W.exact_distances(active)
    pool = W.PoolSpec("syn", cap, [16], np.ones(n, np.uint32))
    tr = W.Trace(f"joint{n}", n, 4, [pool], active, dist, dist.copy(), {})
    run_parity(tr, theta=S, slot_units=8192, ring_slots=2, sample_units=4000,
               label=f"joint sort edge {n}")


@pytest.mark.parametrize("first", [2047, 2048, 2049])
def test_published_list_lengths(first):
    """Plans of 2,048 victims and loads (written to the host by system-scope
    stores), one more and one less, in one step and over victims and loads."""
    n = 6000
    active = np.zeros((5, n), np.uint8)
    active[0, :first] = 1
    for t, k in enumerate((1023, 1024, 1025)):
        active[t + 1, 2100 + 1100 * t:2100 + 1100 * t + k] = 1
    cap = first + 1
    active[4, 3000:3000 + cap] = 1
    dist = W.exact_distances(active)
    pool = W.PoolSpec("syn", cap, [16], np.ones(n, np.uint32))
    tr = W.Trace(f"lists{first}", n, 5, [pool], active, dist, dist.copy(), {})
    mask = (np.random.default_rng(first).random((5, n)) < 0.5).astype(np.uint8)
    for theta in (0, S):
        run_parity(tr, theta=theta, slot_units=8192, ring_slots=2, dirty=mask, check_mirrors=True,
                   label=f"lists {first}, threshold {theta}")
