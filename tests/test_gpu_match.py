"""Matchings of blocks of at most 16 rows: four to a wavefront from some 10,000 blocks on, one to a wavefront below.
Populations that leave the last wavefront with one, two and three candidates, all block sizes at the edges, weights with
many ties and without any, whole evaluations and the trials of the local search, against the oracle to the bit."""
import numpy as np
import pytest

import paper_2206_01288_amd as dtfm
import workloads
from .gpu_util import both, dev, host, oracle_eval_threaded

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ties", [0, 2, 40])
@pytest.mark.parametrize("D_dp,D_pp,P", [(1, 4, 1709), (2, 3, 3415), (3, 9, 289), (7, 8, 367), (8, 5, 1027), (9, 12, 157),
                                         (15, 6, 685), (16, 4, 1710), (16, 16, 87)])
def test_four_blocks_to_a_wavefront(ties, D_dp, D_pp, P):
    N, pairs = D_dp * D_pp, D_pp * (D_pp - 1) // 2
    assert P * pairs > 10240
    rng = np.random.default_rng(1000 * D_dp + D_pp + ties)
    lat = rng.uniform(1e-3, 0.1, (N, N)) if ties == 0 else rng.integers(1, ties + 1, (N, N)) * 0.01
    bw = 10.0 ** rng.uniform(7, 9, (N, N)) if ties == 0 else np.full((N, N), 1e9)
    lat, bw = np.triu(lat, 1) + np.triu(lat, 1).T, np.triu(bw, 1) + np.triu(bw, 1).T
    np.fill_diagonal(bw, 1.0)
    o, g = both(workloads.Workload("match", N, D_dp, D_pp, 1e8, 1e7, lat, bw, 0))
    perms = workloads.random_population(P, N, seed=D_pp)
    cost = host(dtfm.eval_population(g, dev(perms)))
    few = host(dtfm.eval_population(g, dev(perms[:3])))          # one block to a wavefront
    assert np.array_equal(cost[:3], few)
    some = np.arange(P) if D_pp <= 9 else np.r_[0:32, P - 8:P]   # the oracle's full recursion is slow from 12 stages on
    assert np.array_equal(cost[some], oracle_eval_threaded(o, perms[some]))
    if D_dp > 1 and D_pp <= 9:                                   # trials: 2 D_pp - 3 blocks of each of 4 P rows
        last = slice(P - 5, P)
        rows, want, _ = o.local_search(perms[last], 2, dtfm.BEST4)
        rows_d = dev(perms)
        cost_d, _ = dtfm.local_search(g, rows_d, 2, dtfm.BEST4)
        assert np.array_equal(host(rows_d)[last], rows) and np.array_equal(host(cost_d)[last], want)
    dtfm.destroy_problem(g)
