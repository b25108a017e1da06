"""The work a user of this library has it do, as cases that can be timed.

A case names an entry point, a shape (D_dp devices per stage, D_pp stages), a kind of network and a population. The
listed cases follow the benchmark's configurations (the 8-, 64-, 256- and 1024-device problems), the steady-state
mode of the search ablation and one shape that no kernel was tuned for; `draw` spreads over all shapes the library
takes (D_dp <= 64, D_pp <= 16, N <= 1024), odd ones among them, all entry points and the neighbourhoods of the
local search. All results are pinned to the bit (every rounding is defined), so the tolerance is "exact".
"""
import math

import numpy as np
import torch

import paper_2206_01288_amd as dtfm

MS, GBPS = 1e-3, 1e9 / 8.0


def listed():
    return [
        # a unit test's or a notebook's problem: eight devices, one call, nothing but latency
        _case("eval-8dev-p64", "eval", 2, 4, "iid", 64),
        # a shape with no power of two in it, a mid-size population
        _case("eval-84dev-p3001", "eval", 12, 7, "regions", 3001),
        # the headline call: the population of a search on 64 devices, once
        _case("eval-64dev-p4096", "eval", 8, 8, "regions", 4096),
        # the same problem sampled in bulk (random allocations scored to seed or to judge a search)
        _case("eval-64dev-p1048576", "eval", 8, 8, "regions", 1 << 20),
        # 256 devices in 16 stages of 16: the tour over the stages dominates
        _case("eval-256dev-p1024", "eval", 16, 16, "regions", 1024),
        # 1024 devices in 16 stages of 64: the largest problem
        _case("eval-1024dev-p4096", "eval", 64, 16, "clustered", 4096),
        # the paper's loop as written: one offspring at a time, a chain of small launches
        _case("steady-64dev-p256", "evolve", 8, 8, "regions", 256, lam=1, generations=200, moves=8, nb="GAIN4"),
        # the generation-wise search on 64 devices
        _case("evolve-64dev-p4096", "evolve", 8, 8, "regions", 4096, lam=4096, generations=20, moves=8, nb="GAIN4"),
        # the search on 256 devices with all four candidate swaps priced
        _case("evolve-256dev-p1024", "evolve", 16, 16, "regions", 1024, lam=1024, generations=2, moves=2, nb="BEST4"),
        # the search on 1024 devices
        _case("evolve-1024dev-p4096", "evolve", 64, 16, "clustered", 4096, lam=4096, generations=2, moves=8, nb="GAIN4"),
        # exhaustive swap search: 2016 swaps of each of 4096 allocations, 20 rounds
        _case("allpairs-64dev-p4096", "search", 8, 8, "regions", 4096, moves=20, nb="ALL_PAIRS"),
        # the pipelines behind the best allocations of a finished search, ready to deploy
        _case("assign-256dev-p32", "assign", 16, 16, "regions", 32),
    ]


def _case(name, op, D_dp, D_pp, net, P, lam=0, generations=0, moves=0, nb="GAIN4"):
    return {"name": name, "op": op, "D_dp": D_dp, "D_pp": D_pp, "net": net, "P": P, "lam": lam,
            "generations": generations, "moves": moves, "nb": nb}


def draw(rng):
    """One more case of the same ranges. The population is drawn over the logarithm of its range, whose upper end is
    what a rough price of the work leaves room for."""
    while True:
        op = rng.choice(["eval", "eval", "eval", "evolve", "evolve", "search", "search", "assign"])
        if rng.random() < 0.3:
            D_dp, D_pp = 8, 8                      # the shape most searches run on
        else:
            D_pp = rng.randint(2, 16)
            D_dp = min(64, int(round(math.exp(rng.uniform(0.0, math.log(64.49))))))
        N = D_dp * D_pp
        if N < 4 or N > 1024:
            continue
        net = rng.choice(["regions", "regions", "clustered", "clustered", "iid", "tied"])
        nb = "GAIN4"
        lam = generations = moves = 0
        if op == "evolve":
            nb = rng.choice(["GAIN4", "GAIN4", "BEST4", "KL"])
            generations, moves = rng.randint(1, 8), rng.choice([0, 1, 2, 4, 8, 8, 12])
        elif op == "search":
            nb = rng.choice(["GAIN4", "BEST4", "KL", "ALL_PAIRS"])
            moves = rng.randint(1, 3) if nb == "ALL_PAIRS" else rng.randint(1, 12)
        if op in ("evolve", "search") and D_dp < 2 and nb in ("GAIN4", "BEST4"):
            nb = "KL"                              # the four-candidate neighbourhoods need a link inside a stage
        one = _case("", op, D_dp, D_pp, net, 1, 1, generations, moves, nb)
        most = int(min(1 << 20, 2.0e10 / _price(one), 1.0e9 / (4 * N * (5 if op == "evolve" else 2))))
        if op == "search" and nb == "ALL_PAIRS":
            most = min(most, 4096)
        if op == "assign":
            most = min(most, 1024)
        if op == "evolve":
            most = min(most, 16384)
        if most < 2:
            continue
        P = max(1, int(round(math.exp(rng.uniform(0.0, math.log(most))))))
        if op == "evolve":
            lam = rng.choice([P, P, max(1, P // 2), 1])
        c = _case("", op, D_dp, D_pp, net, P, lam, generations, moves, nb)
        del c["name"]
        return c


def _evaluations(c):
    """(full evaluations, trial evaluations of the local search) of one pass, per row of the population."""
    if c["op"] == "evolve":
        per = c["moves"] * (4 if c["nb"] == "BEST4" else 1)
        return 1 + c["generations"], c["generations"] * per
    if c["op"] == "search":
        N = c["D_dp"] * c["D_pp"]
        per = N * (N - 1) // 2 if c["nb"] == "ALL_PAIRS" else 4 if c["nb"] == "BEST4" else 1
        return 1, c["moves"] * per
    return 1, 0


def _price(c):
    """Rough operations of one row: matchings by augmenting paths, Held-Karp over all subsets."""
    n, D = c["D_pp"], c["D_dp"]
    tour = 2.0 * n * (n - 1) * 2.0 ** max(n - 2, 0) * (4.0 if c["op"] == "assign" else 1.0)
    full, trials = _evaluations(c)
    return (full * (n * (n - 1) / 2 * 4.0 * D * D + n * D * D + tour + 2000.0)
            + trials * (2 * n * 4.0 * D * D + n * D * D + tour + 2000.0))


def _network(kind, N, D_pp, rng):
    """(latency in seconds, bandwidth in bytes per second), both N x N and symmetric."""
    if kind == "iid":      # every link of its own
        lat = rng.uniform(1.0, 100.0, (N, N))
        bw = 10.0 ** rng.uniform(-1.0, 1.0, (N, N))
    else:                  # regions of N / R devices, one base value per pair of regions
        R = max(2, min(32, N // 8)) if kind == "clustered" else max(2, min(16, N // 8))
        if kind == "clustered":
            cl = np.arange(R) * 4 // R
            near = cl[:, None] == cl[None, :]
            lat = np.where(near, rng.uniform(10.0, 70.0, (R, R)), rng.uniform(70.0, 250.0, (R, R)))
            bw = np.where(near, rng.uniform(1.0, 1.3, (R, R)), rng.uniform(0.3, 1.3, (R, R)))
            inside = rng.uniform(2.0, 10.0, R)
        else:
            low, high = (0.05, 5.0) if N >= 256 else (0.1, 2.0)
            lat = rng.uniform(20.0, 250.0, (R, R))
            bw = 10.0 ** rng.uniform(math.log10(low), math.log10(high), (R, R))
            inside = rng.uniform(5.0, 10.0, R)
        lat, bw = np.triu(lat, 1) + np.triu(lat, 1).T, np.triu(bw, 1) + np.triu(bw, 1).T
        np.fill_diagonal(lat, rng.uniform(0.5, 5.0, R))
        np.fill_diagonal(bw, inside)
        if kind == "tied":  # printed tables of whole milliseconds and tenths of Gbit/s, the same for all devices of a region
            lat, bw = np.ceil(lat), np.maximum(np.round(bw, 1), 0.1)
        of = np.arange(N) * R // N
        lat, bw = lat[np.ix_(of, of)], bw[np.ix_(of, of)]
        if kind != "tied":  # measured links of one pair of regions differ by some per cent
            lat = lat * rng.uniform(0.95, 1.05, (N, N))
            bw = bw * rng.uniform(0.95, 1.05, (N, N))
    lat, bw = np.triu(lat, 1) + np.triu(lat, 1).T, np.triu(bw, 1) + np.triu(bw, 1).T
    np.fill_diagonal(lat, 1.0)
    np.fill_diagonal(bw, 1.0)
    return lat * MS, bw * GBPS


def prepare(case, seed):
    N, P = case["D_dp"] * case["D_pp"], case["P"]
    lat, bw = _network(case["net"], N, case["D_pp"], np.random.default_rng(seed))
    # gradients of one stage of a 1.3e9-parameter model and activations of one micro-batch hop, 16 bits each
    c_dp, c_pp = 1.3e9 * 2.0 / case["D_pp"], 2048.0 * 2048.0 * 2.0
    prob = dtfm.create_problem(lat, bw, c_dp, c_pp, case["D_dp"], case["D_pp"])
    s = {"case": case, "seed": seed, "prob": prob, "nb": getattr(dtfm, case["nb"])}
    lam = case["lam"] if case["op"] == "evolve" else 0
    dtfm.reserve(prob, P, lam, s["nb"])
    if case["op"] != "evolve":    # evolve makes its own first population
        gen = torch.Generator(device="cuda")
        gen.manual_seed(seed)
        perm = torch.empty((P, N), dtype=torch.int32, device="cuda")
        step = max(1, (1 << 24) // N)
        for p in range(0, P, step):
            n = min(step, P - p)
            perm[p:p + n] = torch.rand((n, N), generator=gen, device="cuda").argsort(dim=1)
        s["perm"] = perm
        s["cost"] = torch.empty(P, dtype=torch.float64, device="cuda")
    if case["op"] == "search":
        s["rows"] = torch.empty_like(perm)
        s["applied"] = torch.empty((P, case["moves"]), dtype=torch.int64, device="cuda")
    return s


def run(s):
    case = s["case"]
    if case["op"] == "eval":
        return dtfm.eval_population(s["prob"], s["perm"], s["cost"])
    if case["op"] == "assign":
        return dtfm.get_assignment(s["prob"], s["perm"])
    if case["op"] == "search":    # in place: on a copy, the caller keeps the rows it started from
        s["rows"].copy_(s["perm"])
        cost, applied = dtfm.local_search(s["prob"], s["rows"], case["moves"], s["nb"], cost=s["cost"], applied=s["applied"])
        return s["rows"], cost, applied
    return dtfm.evolve(s["prob"], s["seed"], case["generations"], case["P"], lam=case["lam"], ls_moves=case["moves"],
                       neighbourhood=s["nb"])


def work(case):
    """Rows read (and written, where the call changes or makes them) once, results written once, the two weight
    matrices read once. Operations: Eq. 2's additions, one look at every entry of every block of Eq. 3 and, for Eq. 4,
    an addition and a minimum per relaxation of the subset recursion up to half the stages (a tour over an undirected
    graph is two half tours that meet). A swap changes two stages: its trial redoes their part of Eqs. 2 and 3."""
    n, D, P = case["D_pp"], case["D_dp"], case["P"]
    N, half = n * D, (n + 1) // 2
    tour = 2.0 * sum(math.comb(n, k) * k * (n - k) for k in range(1, half + 1))
    whole = N * (D - 1.0) + n * (n - 1) / 2.0 * D * D + tour
    trial = 2.0 * D * (D - 1.0) + (2 * n - 3.0) * D * D + tour
    if case["op"] == "search" and case["nb"] == "ALL_PAIRS":
        trial = 4.0 * D + 2.0 * n * D + tour    # one device of each of two stages is new
    bytes_ = 16.0 * N * N
    if case["op"] == "evolve":
        full, trials = _evaluations(case)
        lam, gens = case["lam"], case["generations"]
        bytes_ += 12.0 * P * N + 8.0 * P + 8.0 * lam * N * gens + 8.0 * gens
        return {"bytes": bytes_, "flops": whole * (P + lam * gens) + trial * lam * trials}
    full, trials = _evaluations(case)
    bytes_ += 4.0 * P * N
    if case["op"] == "eval":
        bytes_ += 8.0 * P
    elif case["op"] == "assign":
        bytes_ += 4.0 * P * (N + n)
    else:
        bytes_ += 4.0 * P * N + 8.0 * P + 8.0 * P * case["moves"]
    return {"bytes": bytes_, "flops": P * (whole * full + trial * trials)}


def tolerance(case):
    return "exact"
