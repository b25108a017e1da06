"""Eq. 4 by pruned subset recursion (11 to 16 stages) against the oracle's full recursion, to the bit: unique optima,
ties that widen a layer beyond a wavefront's and a workgroup's tables, equal weights (left to the dense recursion), and
weights over twelve orders of magnitude (the integer bound then resolves next to nothing)."""
import numpy as np
import pytest

import paper_2206_01288_amd as dtfm
import workloads
from .gpu_util import both, dev, host, oracle_eval_threaded

pytestmark = pytest.mark.gpu


def _network(kind, N, rng):
    if kind == "iid":
        lat, bw = rng.uniform(1e-3, 0.1, (N, N)), 10.0 ** rng.uniform(7, 9, (N, N))
    elif kind == "tied":        # three latencies, one bandwidth
        lat, bw = rng.integers(1, 4, (N, N)) * 0.01, np.full((N, N), 1e9)
    elif kind == "equal":
        lat, bw = np.full((N, N), 0.01), np.full((N, N), 1e9)
    else:                       # "range"
        lat, bw = np.zeros((N, N)), 10.0 ** rng.uniform(0, 12, (N, N))
    lat, bw = np.triu(lat, 1) + np.triu(lat, 1).T, np.triu(bw, 1) + np.triu(bw, 1).T
    np.fill_diagonal(bw, 1.0)
    return lat, bw


@pytest.mark.parametrize("kind", ["iid", "tied", "equal", "range"])
@pytest.mark.parametrize("D_dp,D_pp,P", [(1, 11, 1), (2, 11, 7), (3, 12, 9), (2, 13, 6), (3, 14, 5), (1, 15, 3), (1, 16, 2), (4, 16, 6)])
def test_pruned_tour(kind, D_dp, D_pp, P):
    N = D_dp * D_pp
    rng = np.random.default_rng(100 * D_pp + D_dp)
    lat, bw = _network(kind, N, rng)
    o, g = both(workloads.Workload("tour", N, D_dp, D_pp, 1e8, 1e7, lat, bw, 0))
    perms = workloads.random_population(P, N, seed=D_pp)
    want = oracle_eval_threaded(o, perms)
    assert np.array_equal(host(dtfm.eval_population(g, dev(perms))), want)
    order, sigma = dtfm.get_assignment(g, dev(perms))
    for p in range(min(P, 3)):
        order_o, sigma_o = o.get_assignment(perms[p])
        assert np.array_equal(host(order)[p], order_o) and np.array_equal(host(sigma)[p], sigma_o)
    if D_dp > 1:                # trials with a cost to beat, the search that follows from them
        for nb in (dtfm.KL, dtfm.BEST4):
            rows, cost, applied = o.local_search(perms, 3, nb)
            rows_d = dev(perms)
            applied_d = dev(np.empty((P, 3), dtype=np.int64))
            cost_d, _ = dtfm.local_search(g, rows_d, 3, nb, applied=applied_d)
            assert np.array_equal(host(rows_d), rows) and np.array_equal(host(cost_d), cost) and np.array_equal(host(applied_d), applied)
    dtfm.destroy_problem(g)
