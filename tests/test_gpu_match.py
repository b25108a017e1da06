"""Matchings of blocks of 9 to 16 rows: four to a wavefront from 1536 blocks for each row on, one to a wavefront below; of at most
8 rows a lane for two, few of them one to a wavefront; of more on bit masks or by smallest entries. Populations that leave the last
wavefront with one, two and three candidates, all block sizes at the edges, weights with many ties and without any, whole
evaluations and the trials of the local search, against the oracle to the bit."""
import numpy as np
import pytest
import torch

import paper_2206_01288_amd as dtfm
import workloads
from .gpu_util import both, dev, host, oracle_eval_threaded

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ties", [0, 2, 40])
@pytest.mark.parametrize("D_dp,D_pp,P", [(1, 4, 1709), (2, 3, 3415), (3, 9, 289), (7, 8, 387), (8, 5, 1231), (9, 12, 213), (10, 3, 5121),
                                         (11, 9, 470), (13, 8, 714), (15, 6, 1537), (16, 4, 4098), (16, 16, 207)])
def test_many_blocks_of_at_most_16_rows(ties, D_dp, D_pp, P):
    # 9 to 16 rows: four blocks to a wavefront, the first rows alone one to a wavefront; fewer rows: two to a lane
    N, pairs = D_dp * D_pp, D_pp * (D_pp - 1) // 2
    assert P * pairs > max(10240, 1536 * D_dp) and (D_dp <= 8 or 3 * pairs <= 1536 * D_dp)
    rng = np.random.default_rng(1000 * D_dp + D_pp + ties)
    lat = rng.uniform(1e-3, 0.1, (N, N)) if ties == 0 else rng.integers(1, ties + 1, (N, N)) * 0.01
    bw = 10.0 ** rng.uniform(7, 9, (N, N)) if ties == 0 else np.full((N, N), 1e9)
    lat, bw = np.triu(lat, 1) + np.triu(lat, 1).T, np.triu(bw, 1) + np.triu(bw, 1).T
    np.fill_diagonal(bw, 1.0)
    o, g = both(workloads.Workload("match", N, D_dp, D_pp, 1e8, 1e7, lat, bw, 0))
    perms = workloads.random_population(P, N, seed=D_pp)
    cost = host(dtfm.eval_population(g, dev(perms)))
    graphs = host(dtfm.coarsened_graph(g, dev(perms))[0])
    assert np.array_equal(graphs[:3], host(dtfm.coarsened_graph(g, dev(perms[:3]))[0]))
    some = np.arange(P) if D_pp <= 9 else np.r_[0:32, P - 8:P]   # the oracle's full recursion is slow from 12 stages on
    assert np.array_equal(cost[some], oracle_eval_threaded(o, perms[some]))
    if D_dp > 1 and D_pp <= 9:                                   # trials: 2 D_pp - 3 blocks of each of 4 P rows
        last = slice(P - 5, P)
        rows, want, _ = o.local_search(perms[last], 2, dtfm.BEST4)
        rows_d = dev(perms)
        cost_d, _ = dtfm.local_search(g, rows_d, 2, dtfm.BEST4)
        assert np.array_equal(host(rows_d)[last], rows) and np.array_equal(host(cost_d)[last], want)
    dtfm.destroy_problem(g)


@pytest.mark.parametrize("D_dp,D_pp,P", [(9, 12, 213), (16, 12, 373), (13, 16, 167), (16, 16, 207)])
def test_four_blocks_to_a_wavefront_of_many_stages(D_dp, D_pp, P):
    # every edge of the graphs themselves, and of trials that start from other graphs (2 D_pp - 3 blocks of a row; the
    # graph of the accepted row carries them on)
    N = D_dp * D_pp
    rng = np.random.default_rng(D_dp)
    lat, bw = rng.integers(1, 400, (N, N)) * 1e-4, np.full((N, N), 1e9)
    lat, bw = np.triu(lat, 1) + np.triu(lat, 1).T, np.triu(bw, 1) + np.triu(bw, 1).T
    np.fill_diagonal(bw, 1.0)
    o, g = both(workloads.Workload("match", N, D_dp, D_pp, 1e7, 1e7, lat, bw, 0))
    perms = workloads.random_population(P, N, seed=D_pp)
    ghat, _ = dtfm.coarsened_graph(g, dev(perms))
    ghat = host(ghat)
    for p in np.r_[0:24, P - 24:P]:
        assert np.array_equal(ghat[p], o.coarsen(perms[p])), p
    many = np.concatenate([perms] * 6)
    assert len(many) * (2 * D_pp - 3) > 1536 * D_dp
    rows, want, _ = o.local_search(perms[-3:], 3, dtfm.KL)
    rows_d = dev(many)
    cost_d, _ = dtfm.local_search(g, rows_d, 3, dtfm.KL)
    assert np.array_equal(host(rows_d)[-3:], rows) and np.array_equal(host(cost_d)[-3:], want)
    dtfm.destroy_problem(g)


@pytest.mark.parametrize("D_dp,D_pp,blocks", [(9, 12, 1536 * 9), (12, 7, 1536 * 12), (16, 3, 1536 * 16), (17, 4, 32768), (18, 8, 32768), (19, 8, 32768)])
def test_no_jump_where_the_kernel_changes(D_dp, D_pp, blocks):
    # one per cent more rows on the other side cost at most a tenth more
    N, pairs = D_dp * D_pp, D_pp * (D_pp - 1) // 2
    w = workloads.Workload("match", N, D_dp, D_pp, 1e8, 1e7, *workloads.network_regions(N // 4, 4, seed=1), 0)
    g = dtfm.create_problem(w.latency, w.bandwidth, w.c_dp, w.c_pp, D_dp, D_pp)
    below = blocks // pairs
    perms = dev(workloads.random_population(below + below // 100 + 1, N, seed=2))
    best = {}
    for _ in range(8):
        for P in (below, len(perms)):
            rows, out = perms[:P], torch.empty(P, dtype=torch.float64, device="cuda")
            dtfm.eval_population(g, rows, out)
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(10):
                dtfm.eval_population(g, rows, out)
            b.record()
            torch.cuda.synchronize()
            best[P] = min(best.get(P, np.inf), a.elapsed_time(b))
    assert best[len(perms)] <= 1.1 * best[below], best
    dtfm.destroy_problem(g)


@pytest.mark.parametrize("D_dp,D_pp,P", [(17, 3, 9), (31, 4, 40), (32, 3, 700), (33, 4, 9), (47, 3, 40), (63, 4, 3), (64, 4, 40),
                                         (64, 2, 900), (18, 3, 10930), (19, 5, 3277), (24, 2, 7), (32, 2, 2048), (33, 3, 2740), (48, 2, 8193)])
@pytest.mark.parametrize("kind", ["equal", "few", "thousand", "all", "near"])
def test_blocks_of_more_than_16_rows(kind, D_dp, D_pp, P):
    # the last six: many blocks, which go by smallest entries on all networks (18 and 19 rows) or on those whose links are all of their
    # own (all). Ranks of one digit (2 and 61 weights), two (1000) and three (16,130 and more); near: the blocks between two halves of
    # the network hold weights of neighbouring ranks only, so that columns hold many entries of the optimum's leading digit
    N = D_dp * D_pp
    rng = np.random.default_rng(100 * D_dp + D_pp)
    lat = {"equal": np.full((N, N), 0.01), "few": rng.integers(1, 62, (N, N)) * 1e-3,
           "thousand": rng.integers(1, 1001, (N, N)) * 1e-4}.get(kind, rng.uniform(1e-3, 0.1, (N, N)))
    if kind == "near":
        far = (np.arange(N)[:, None] < N // 2) != (np.arange(N)[None, :] < N // 2)
        lat = np.where(far, 0.05 + 1e-7 * rng.uniform(0.0, 1.0, (N, N)), lat)
    lat = np.triu(lat, 1) + np.triu(lat, 1).T
    bw = np.full((N, N), 1e9)
    o, g = both(workloads.Workload("match", N, D_dp, D_pp, 1e7, 1e7, lat, bw, 0))
    perms = workloads.random_population(P, N, seed=D_pp)
    perms[0] = np.arange(N)              # stages that lie in one half each
    perms[1] = np.arange(N)[::-1]
    ghat = host(dtfm.coarsened_graph(g, dev(perms))[0])
    some = np.r_[0:min(P, 6), max(P - 3, 0):P]
    for p in some:
        assert np.array_equal(ghat[p], o.coarsen(perms[p])), p
    if D_pp > 2:                          # trials: the 2 D_pp - 3 blocks of a round's two stages
        rows, want, _ = o.local_search(perms[some], 3, dtfm.KL)
        rows_d = dev(perms)
        cost_d, _ = dtfm.local_search(g, rows_d, 3, dtfm.KL)
        assert np.array_equal(host(rows_d)[some], rows) and np.array_equal(host(cost_d)[some], want)
    dtfm.destroy_problem(g)


@pytest.mark.parametrize("D_dp,D_pp", [(1, 1), (5, 1), (1, 2), (16, 2), (2, 4), (8, 5), (16, 5), (1, 6), (16, 6)])
@pytest.mark.parametrize("ties", [0, 3])
def test_small_evaluations_in_one_launch(ties, D_dp, D_pp):
    # 512 rows of 5 stages and 256 of 6 in one launch, one more in three; searches whose rounds take one launch too
    N, most = D_dp * D_pp, 512 if D_pp <= 5 else 256
    rng = np.random.default_rng(D_dp + 100 * D_pp)
    lat = rng.uniform(1e-3, 0.1, (N, N)) if ties == 0 else rng.integers(1, ties + 1, (N, N)) * 0.01
    lat, bw = np.triu(lat, 1) + np.triu(lat, 1).T, np.full((N, N), 1e9)
    o, g = both(workloads.Workload("small", N, D_dp, D_pp, 1e8, 1e7, lat, bw, 0))
    perms = workloads.random_population(most + 1, N, seed=D_pp)
    want = oracle_eval_threaded(o, perms)
    for P in (1, 7, most, most + 1):
        assert np.array_equal(host(dtfm.eval_population(g, dev(perms[:P]))), want[:P])
    if D_dp > 1 and D_pp > 1:
        for nb, P in ((dtfm.GAIN4, 9), (dtfm.KL, most), (dtfm.BEST4, most // 4), (dtfm.BEST4, most // 4 + 1), (dtfm.ALL_PAIRS, 2)):
            moves = 1 if nb == dtfm.ALL_PAIRS else 3
            rows, cost, _ = o.local_search(perms[:P], moves, nb)
            rows_d = dev(perms[:P])
            cost_d, _ = dtfm.local_search(g, rows_d, moves, nb)
            assert np.array_equal(host(rows_d), rows) and np.array_equal(host(cost_d), cost)
    dtfm.destroy_problem(g)


@pytest.mark.parametrize("D_dp,D_pp,P", [(1, 7, 1), (2, 7, 3), (3, 7, 171), (4, 8, 2), (5, 11, 40), (6, 9, 700), (7, 8, 5), (8, 7, 90),
                                         (8, 16, 140), (8, 16, 32), (8, 16, 33), (7, 14, 28), (7, 14, 29), (6, 16, 10), (6, 16, 11), (8, 9, 14), (8, 9, 15)])
@pytest.mark.parametrize("ties", [0, 3])
def test_two_blocks_to_a_lane(ties, D_dp, D_pp, P):
    # odd and even numbers of stage pairs (the odd one out is matched twice) and of trial pairs; 16 x 8: codes up to 8130; the last
    # eight: numbers of blocks on both sides of the line below which a block has a wavefront
    N = D_dp * D_pp
    rng = np.random.default_rng(D_dp + 100 * D_pp)
    lat = rng.uniform(1e-3, 0.1, (N, N)) if ties == 0 else rng.integers(1, ties + 1, (N, N)) * 0.01
    lat, bw = np.triu(lat, 1) + np.triu(lat, 1).T, np.full((N, N), 1e9)
    o, g = both(workloads.Workload("lanes", N, D_dp, D_pp, 1e8, 1e7, lat, bw, 0))
    perms = workloads.random_population(P, N, seed=D_pp)
    ghat = host(dtfm.coarsened_graph(g, dev(perms))[0])
    some = np.r_[0:min(P, 6), max(P - 3, 0):P]
    for p in some:
        assert np.array_equal(ghat[p], o.coarsen(perms[p])), p
    rows, want, _ = o.local_search(perms[some], 2, dtfm.KL)
    rows_d = dev(perms)
    cost_d, _ = dtfm.local_search(g, rows_d, 2, dtfm.KL)
    assert np.array_equal(host(rows_d)[some], rows) and np.array_equal(host(cost_d)[some], want)
    dtfm.destroy_problem(g)


@pytest.mark.parametrize("D_dp", [48, 64])
def test_links_of_their_own_take_no_longer(D_dp):
    # every link of its own: optima of small digits, which a descent from a larger one reaches by losing most of the matching
    N, P = 8 * D_dp, 1000
    rng = np.random.default_rng(D_dp)
    best = {}
    perms = dev(workloads.random_population(P, N, seed=1))
    for kind in ("own", "regions"):
        lat = rng.uniform(1e-3, 0.1, (N, N))
        if kind == "regions":
            of = np.arange(N) * 8 // N
            lat = rng.uniform(0.02, 0.25, (8, 8))[np.ix_(of, of)] * rng.uniform(0.95, 1.05, (N, N))
        lat = np.triu(lat, 1) + np.triu(lat, 1).T
        g = dtfm.create_problem(lat, np.full((N, N), 1e9), 1e7, 1e7, D_dp, 8)
        out = dtfm.coarsened_graph(g, perms)
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(10):
                dtfm.coarsened_graph(g, perms, out=out)
            b.record()
            b.synchronize()
            best[kind] = min(best.get(kind, np.inf), a.elapsed_time(b))
        dtfm.destroy_problem(g)
    assert best["own"] <= 1.25 * best["regions"], best


@pytest.mark.parametrize("D_dp,D_pp,below,moves", [(2, 4, 512, None), (8, 5, 512, None), (16, 5, 512, None), (16, 6, 256, None), (16, 16, 1024, None),
                                                   (4, 13, 1024, None), (1, 14, 512, None), (8, 16, 32, None), (8, 8, 256, 1),
                                                   (8, 8, 256, 4), (8, 8, 256, 8)])
def test_few_rows_take_no_longer_than_more(D_dp, D_pp, below, moves):
    # launches of few rows go ways of their own up to a line (evaluation in one launch, lone tours, wavefronts for blocks of 8 rows,
    # rounds priced ahead): never more time there than for a row, or a tenth of the rows, beyond it
    N = D_dp * D_pp
    w = workloads.Workload("few", N, D_dp, D_pp, 1e8, 1e7, *workloads.network_iid(N, seed=1), 0)
    g = dtfm.create_problem(w.latency, w.bandwidth, w.c_dp, w.c_pp, D_dp, D_pp)
    perms = dev(workloads.random_population(below + 1 if moves else below + below // 10, N, seed=2))
    best = {}
    for P in (below, len(perms)):
        rows, out = perms[:P].clone(), torch.empty(P, dtype=torch.float64, device="cuda")

        def call():
            if moves:
                dtfm.local_search(g, rows, moves, dtfm.GAIN4, cost=out)
            else:
                dtfm.eval_population(g, rows, out)

        call()
        for _ in range(8):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(20):
                call()
            b.record()
            torch.cuda.synchronize()
            best[P] = min(best.get(P, np.inf), a.elapsed_time(b) / 20)
    assert best[below] <= 1.1 * best[len(perms)] + 0.001, best
    dtfm.destroy_problem(g)
