"""Plan kernels at the edges of their agent counts and sorted sets, against the
oracle's plans and bytes."""
import numpy as np
import pytest

import workloads as W
from gpu_harness import S, run_parity

pytestmark = pytest.mark.gpu


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
