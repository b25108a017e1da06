"""Eq. 4 from 11 stages on, by pruned subset recursion and by the dense one, against the oracle's full recursion, to the bit:
unique optima, ties that widen a layer beyond a wavefront's and a workgroup's tables, equal weights (answered at once),
weights over twelve orders of magnitude (the integer bound then resolves next to nothing), weights whose sums the pruned
recursion leaves to the dense one whatever the graph, and launches of all sizes at which rows change their route."""
import numpy as np
import pytest
import torch

import paper_2206_01288_amd as dtfm
import workloads
from .gpu_util import both, dev, host, oracle_eval_threaded

pytestmark = pytest.mark.gpu


TINY = 1e-290   # bytes: costs of 1e-298 s and up, below what the pruned recursion takes


def _network(kind, N, rng):
    if kind == "iid":
        lat, bw = rng.uniform(1e-3, 0.1, (N, N)), 10.0 ** rng.uniform(7, 9, (N, N))
    elif kind == "tied":        # three latencies, one bandwidth
        lat, bw = rng.integers(1, 4, (N, N)) * 0.01, np.full((N, N), 1e9)
    elif kind == "two":         # sites of eight devices
        same = np.arange(N)[:, None] // 8 == np.arange(N) // 8
        lat, bw = np.where(same, 1e-3, 5e-2), np.where(same, 1.25e9, 1.25e8)
    elif kind == "twenty":      # whole milliseconds
        lat, bw = rng.integers(1, 21, (N, N)) * 1e-3, np.full((N, N), 1e9)
    elif kind in ("tiny", "zero"):
        lat, bw = np.zeros((N, N)), 10.0 ** rng.uniform(7, 9, (N, N))
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


def _problems(kind, D_dp, D_pp, seed):
    lat, bw = _network(kind, D_dp * D_pp, np.random.default_rng(seed))
    c = {"tiny": (TINY, TINY), "zero": (1e8, 0.0)}.get(kind, (1e8, 1e7))
    return both(workloads.Workload("tour", D_dp * D_pp, D_dp, D_pp, c[0], c[1], lat, bw, 0))


@pytest.mark.parametrize("kind", ["tiny", "zero"])
@pytest.mark.parametrize("D_dp,D_pp,P", [(2, 11, 2400), (2, 12, 1400), (2, 13, 900), (2, 14, 300), (2, 16, 300), (1, 15, 20)])
def test_dense_recursion(kind, D_dp, D_pp, P):
    # every row of these goes through the list of the dense recursion, more of them than it has workgroups
    N = D_dp * D_pp
    o, g = _problems(kind, D_dp, D_pp, D_pp)
    perms = workloads.random_population(P, N, seed=D_pp)
    rows_d = dev(perms)
    cost = host(dtfm.eval_population(g, rows_d))
    some = np.r_[0:P:max(1, P // 150), P - 5:P]
    assert np.array_equal(cost[some], oracle_eval_threaded(o, perms[some]))
    assert np.array_equal(host(dtfm.eval_population_noalloc(g, rows_d, torch.empty(P, dtype=torch.float64, device="cuda"))), cost)
    assert np.array_equal(np.concatenate([host(dtfm.eval_population(g, dev(perms[p:p + 16]))) for p in range(0, P, 16)]), cost)
    order, sigma = dtfm.get_assignment(g, dev(perms[:40]))
    for p in (0, 1, 39 if P > 39 else P - 1):
        order_o, sigma_o = o.get_assignment(perms[p])
        assert np.array_equal(host(order)[p], order_o) and np.array_equal(host(sigma)[p], sigma_o)
    last = slice(P - 4, P)
    for nb in (dtfm.KL, dtfm.BEST4) if D_dp > 1 else ():
        rows, want, _ = o.local_search(perms[last], 2, nb)
        rows_d = dev(perms)
        cost_d, _ = dtfm.local_search(g, rows_d, 2, nb)
        assert np.array_equal(host(rows_d)[last], rows) and np.array_equal(host(cost_d)[last], want)
    dtfm.destroy_problem(g)


@pytest.mark.parametrize("kind", ["iid", "tied", "two", "twenty"])
@pytest.mark.parametrize("D_dp,D_pp", [(4, 11), (2, 12), (16, 12), (4, 13), (2, 14), (16, 14), (4, 15), (1, 16), (16, 16)])
def test_rows_in_launches_of_all_sizes(kind, D_dp, D_pp):
    # a row is searched by a wavefront, by a workgroup or densely by the size of its launch and the values of its edges
    # and of the others': its cost is the same. Sizes around one, two, four and sixteen rounds of 256 rows and the
    # thresholds of 11 to 13 stages.
    N, P = D_dp * D_pp, 4200
    o, g = _problems(kind, D_dp, D_pp, 10 * D_pp + D_dp)
    perms = workloads.random_population(P, N, seed=D_pp)
    rows_d = dev(perms)
    cost = host(dtfm.eval_population(g, rows_d))
    some = np.r_[0:16, P - 16:P]
    assert np.array_equal(cost[some], oracle_eval_threaded(o, perms[some]))
    for n in (1, 8, 9, 255, 256, 257, 513, 769, 1025, 1281, 2049, 2305):
        assert np.array_equal(host(dtfm.eval_population(g, rows_d[P - n:].contiguous())), cost[P - n:]), n
    out = torch.empty(P, dtype=torch.float64, device="cuda")
    assert np.array_equal(host(dtfm.eval_population_noalloc(g, rows_d, out)), cost)
    if D_dp > 1:
        for n, nb in ((3, dtfm.KL), (300, dtfm.BEST4), (1100, dtfm.KL)):
            rows, want, _ = o.local_search(perms[n - 2:n], 2, nb)
            part = dev(perms[:n])
            cost_d, _ = dtfm.local_search(g, part, 2, nb)
            assert np.array_equal(host(part)[n - 2:], rows) and np.array_equal(host(cost_d)[n - 2:], want)
    dtfm.destroy_problem(g)


def _microseconds(g, rows):
    out = torch.empty(len(rows), dtype=torch.float64, device="cuda")
    best = np.inf
    for _ in range(8):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(5):
            dtfm.eval_population(g, rows, out)
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) * 200.0)
    return best


@pytest.mark.parametrize("kind,D_dp,D_pp,P", [("two", 4, 11, 64), ("iid", 4, 11, 1024), ("iid", 2, 12, 64), ("tied", 4, 13, 256),
                                              ("tied", 2, 14, 64), ("tied", 4, 16, 64), ("twenty", 16, 16, 64)])
def test_a_row_is_not_paid_for_twice(kind, D_dp, D_pp, P):
    # where the pruned recursion does not pay, an evaluation takes what it takes by the dense recursion (the weights
    # of "tiny"): five per cent more and two launches are left to it, and as much again to the clock
    rows = dev(workloads.random_population(P, D_dp * D_pp, seed=3))
    _, g = _problems(kind, D_dp, D_pp, 5)
    _, base = _problems("tiny", D_dp, D_pp, 5)
    t, t_base = _microseconds(g, rows), _microseconds(base, rows)
    assert t <= 1.1 * t_base + 16.0, (t, t_base)
    dtfm.destroy_problem(g)
    dtfm.destroy_problem(base)
