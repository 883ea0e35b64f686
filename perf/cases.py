"""The work this framework is asked to do, as cases to time.

A case is a dict of plain values.  `listed()` gives the named ones, `draw(rng)`
one more of the same ranges, `prepare(case, seed)` what a program holds before
the call (device inputs, outputs, workspace or plan), `run(state)` one pass
through the public entry points, `work(case)` the bytes and operations a pass
cannot do without, and `exact(case, seed)` the same outputs from a plain
64-bit evaluation of the recursions' definitions.

Inputs follow paper_2602_05179_amd/workloads.py (integer coordinates on a
grid, rounded Euclidean costs, demands round(Normal(mu, 0.3 mu)) >= 1 with
mu ~ U{1..mu_hi}, uniform or Poisson where that module uses them); only the
demand matrix is drawn on the GPU, because it is large.

Kinds:
  eval       one giant tour on S scenarios (split_eval_device)
  batch      ragged candidate tours sharing the scenarios (Plan.launch)
  routes     route recovery of one tour (split_routes_device)
  variant    overload penalty and/or fleet bound (split_variant_device)
  values     the full value table of one tour (split_values_device)
  inventory  order-up-to DP and its decisions (ou_dp, or the generator and
             the generic update past its 31 levels, then minplus_backtrack)
"""
import math

import numpy as np
import torch

from paper_2602_05179_amd import binding
from paper_2602_05179_amd import workloads as W

DEV = "cuda:0"
INF = int(binding.SPLIT_INF)
BIG = 1 << 40  # "no split" inside exact(): above every finite total


def listed():
    return [
        # one small evaluation inside a heuristic's inner loop: latency
        {"name": "eval_small", "kind": "eval", "n": 20, "N": 20, "S": 1000, "Q": 30, "law": "uniform", "mu_hi": 10},
        # one candidate tour on the usual scenario set of a search
        {"name": "eval_medium", "kind": "eval", "n": 100, "N": 100, "S": 100_000, "Q": 100, "law": "normal", "mu_hi": 20},
        # the headline evaluation: the paper's scale
        {"name": "eval_paper", "kind": "eval", "n": 200, "N": 200, "S": 1_000_000, "Q": 150, "law": "normal", "mu_hi": 20},
        # the longest tours of the request stream, with its largest vehicles
        {"name": "eval_pool", "kind": "eval", "n": 1000, "N": 1000, "S": 20_000, "Q": 300, "law": "normal", "mu_hi": 20},
        # demands in fine units (kilograms): past a byte, ordinary routes
        {"name": "eval_units", "kind": "eval", "n": 150, "N": 150, "S": 100_000, "Q": 3000, "law": "normal", "mu_hi": 400},
        # parcel rounds: small demands, about a hundred stops to a vehicle
        {"name": "eval_parcel", "kind": "eval", "n": 300, "N": 300, "S": 20_000, "Q": 200, "law": "normal", "mu_hi": 3},
        # one generation of a genetic search: ragged candidates in one replay
        {"name": "batch_generation", "kind": "batch", "T": 256, "n_lo": 50, "n_hi": 400, "S": 10_000, "Q": 100},
        # the routes of every scenario, for a plan that is to be carried out
        {"name": "routes_plan", "kind": "routes", "n": 200, "N": 200, "S": 200_000, "Q": 150, "law": "normal", "mu_hi": 20},
        # soft capacity: each vehicle pays for its overload
        {"name": "variant_soft", "kind": "variant", "n": 200, "N": 200, "S": 200_000, "Q": 150, "law": "normal",
         "mu_hi": 20, "beta": 10, "K": 0},
        # hard capacity and a fleet of 25 vehicles (20.6 routes on average)
        {"name": "variant_fleet", "kind": "variant", "n": 200, "N": 200, "S": 200_000, "Q": 150, "law": "normal",
         "mu_hi": 20, "beta": -1, "K": 25},
        # every prefix value of every scenario, for inspecting a tour
        {"name": "values_table", "kind": "values", "n": 100, "N": 100, "S": 100_000, "Q": 100, "law": "normal", "mu_hi": 20},
        # reinsertion decisions of 100 customers in 1000 scenarios, one week
        {"name": "inventory_week", "kind": "inventory", "customers": 100, "scenarios": 1000, "U": 20, "T": 7, "R": 4},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _tour_case(rng, kind, most, stops_lo, stops_hi, mus, n_hi=1000, s_hi=1_000_000):
    """n, N, S, Q of a one-tour case with at most `most` demands: vehicles
    that take stops_lo..stops_hi customers of mean demand (mu_hi + 1) / 2."""
    n = _log_int(rng, 20, n_hi)
    N = n if rng.random() < 0.75 else int(round(n * rng.uniform(1.0, 2.0)))
    mu_hi = mus[rng.randrange(len(mus))]
    S = _log_int(rng, 1000, max(1000, min(s_hi, most // N)))
    Q = max(mu_hi + 1, int(round(rng.uniform(stops_lo, stops_hi) * (mu_hi + 1) / 2)))
    return {"kind": kind, "n": n, "N": N, "S": S, "Q": Q, "law": "normal", "mu_hi": mu_hi}


def draw(rng):
    x = rng.random()
    if x < 0.30:  # byte demands, the request stream's vehicles (4 to 30 stops)
        return _tour_case(rng, "eval", 200_000_000, 5, 30, (20,))
    if x < 0.38:  # fine units
        return _tour_case(rng, "eval", 15_000_000, 5, 25, (200, 400, 1000), n_hi=400, s_hi=100_000)
    if x < 0.45:  # parcel rounds
        return _tour_case(rng, "eval", 4_000_000, 40, 120, (3, 5), n_hi=400, s_hi=20_000)
    if x < 0.55:
        n_hi = _log_int(rng, 60, 400)
        return {"kind": "batch", "T": _log_int(rng, 8, 256), "n_lo": max(10, n_hi // rng.randint(1, 8)), "n_hi": n_hi,
                "S": _log_int(rng, 1000, 10_000), "Q": rng.randint(60, 200)}
    if x < 0.67:
        return _tour_case(rng, "routes", 40_000_000, 5, 30, (20,), n_hi=600, s_hi=200_000)
    if x < 0.82:
        c = _tour_case(rng, "variant", 20_000_000, 6, 18, (20,), n_hi=400, s_hi=200_000)
        hard = rng.random() < 0.5
        c["beta"] = -1 if hard else rng.choice((1, 5, 10, 25))
        least = c["n"] * 10.5 / c["Q"]  # vehicles that the mean demand fills
        c["K"] = int(math.ceil(least * rng.uniform(1.1, 1.6))) if hard or rng.random() < 0.4 else 0
        return c
    if x < 0.90:
        return _tour_case(rng, "values", 10_000_000, 5, 25, (20,), n_hi=400, s_hi=100_000)
    return {"kind": "inventory", "customers": rng.randint(10, 100), "scenarios": _log_int(rng, 100, 1000),
            "U": rng.randint(7, 31) if rng.random() < 0.6 else rng.randint(32, 48), "T": rng.randint(3, 10),
            "R": rng.randint(2, 8)}


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _demands(case, seed, mu, N, S):
    """int16 [S, N] on the GPU, drawn in chunks of about 32M values."""
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 7919 + 17)
    out = torch.empty((S, N), dtype=torch.int16, device=DEV)
    law = case.get("law", "poisson")
    m = torch.as_tensor(mu, dtype=torch.float32, device=DEV)
    step = max(1, (1 << 25) // N)
    for s0 in range(0, S, step):
        rows = min(step, S - s0)
        if law == "uniform":
            x = torch.randint(1, case["mu_hi"] + 1, (rows, N), device=DEV, generator=g)
        elif law == "normal":
            x = torch.randn((rows, N), device=DEV, generator=g)
            x = x.mul_(0.3).add_(1.0).mul_(m).round_().clamp_(1, 32767)
        else:
            x = torch.poisson(m.expand(rows, N), generator=g).clamp_(1, 32767)
        out[s0:s0 + rows] = x.to(torch.int16)
    return out


def _dev(a, dtype):
    return torch.from_numpy(np.ascontiguousarray(a, dtype)).to(DEV)


def _tour_inputs(case, seed):
    rng = np.random.default_rng(int(seed))
    n, N = case["n"], case["N"]
    dist = W.dist_round(W.coords(rng, N))
    tour = W.random_tour(rng, N)[:n]
    mu = rng.integers(1, case["mu_hi"] + 1, size=N)
    return dict(tour=_dev(tour, np.int32), dist=_dev(dist, np.int32), dem=_demands(case, seed, mu, N, case["S"]))


def _batch_inputs(case, seed):
    rng = np.random.default_rng(int(seed))
    N = case["n_hi"]
    dist = W.dist_round(W.coords(rng, N))
    mu = rng.uniform(2.0, 15.0, size=N)
    base = W.random_tour(rng, N)
    tours, lens = [], []
    for t in range(case["T"]):
        k = int(rng.integers(case["n_lo"], case["n_hi"] + 1))
        cand = W.random_tour(rng, k) if t % 2 == 0 else base[base <= k]
        tours.append(W.two_opt_perturb(rng, cand, int(rng.integers(0, 21))))
        lens.append(k)
    return dict(tours=_dev(np.concatenate(tours), np.int32), lens=_dev(lens, np.int32), dist=_dev(dist, np.int32),
                dem=_demands(case, seed, mu, N, case["S"]))


def _inventory_inputs(case, seed):
    rng = np.random.default_rng(int(seed))
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 7919 + 29)
    U, T, R = case["U"], case["T"], case["R"]
    B = case["customers"] * case["scenarios"]
    lam = np.repeat(rng.uniform(1.0, max(1.0, U / 3.0), size=case["customers"]), case["scenarios"])
    lam = torch.as_tensor(lam, dtype=torch.float32, device=DEV)
    demand = torch.poisson(lam.expand(T, B), generator=g).clamp_(max=U + 2).to(torch.int32)
    hold = int(round(float(rng.integers(1, 6, size=case["customers"]).mean())))
    cost = torch.randint(5, 61, (T, B, R), device=DEV, generator=g, dtype=torch.int32)
    cap = torch.randint(0, U + 1, (T, B, R), device=DEV, generator=g, dtype=torch.int32)
    start = _dev(np.repeat(rng.integers(0, U + 1, size=case["customers"]), case["scenarios"]), np.int64)
    J0 = torch.full((B, U + 1), int(binding.MINPLUS_INF), dtype=torch.int32, device=DEV)
    J0[torch.arange(B, device=DEV), start] = 0
    return dict(demand=demand, cost=cost, cap=cap, h=_dev(hold * np.arange(U + 1), np.int32), u=1, rho=4 * hold, J0=J0)


def _scratch(nbytes):
    return torch.empty(max(int(nbytes), 256), dtype=torch.uint8, device=DEV)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "inventory":
        s = _inventory_inputs(case, seed)
        U, T, B = case["U"], case["T"], s["J0"].shape[0]
        if U <= 31:
            s["out"] = (torch.empty((B, U + 1), dtype=torch.int32, device=DEV),
                        torch.empty((T, B, U + 1), dtype=torch.int32, device=DEV))
        else:
            s["A"] = torch.empty((T, B, U + 1, U + 1), dtype=torch.int32, device=DEV)
    elif kind == "batch":
        s = _batch_inputs(case, seed)
        s["plan"] = binding.Plan(s["tours"], s["lens"], s["dist"], s["dem"], case["Q"], max_len=case["n_hi"])
    else:
        s = _tour_inputs(case, seed)
        n, N, S = case["n"], case["N"], case["S"]
        if kind == "eval":
            s["lens"] = _dev([n], np.int32)
            s["out"] = binding.DeviceOutputs(1, S, DEV)
            s["ws"] = _scratch(binding.workspace_bytes(1, n, N, S, case["Q"]))
        elif kind == "routes":
            s["out"] = binding.RouteOutputs(n, S, DEV)
            s["out"].cuts.zero_()  # entries past a scenario's route count are not written
            s["ws"] = _scratch(binding.routes_workspace_bytes(n, N, S))
        elif kind == "variant":
            s["out"] = binding.VariantOutputs(S, DEV)
            s["ws"] = _scratch(binding.variant_workspace_bytes(n, N, S, case["K"]))
        else:
            s["out"] = (torch.empty((n, S), dtype=torch.int32, device=DEV),
                        torch.empty(1, dtype=torch.int32, device=DEV))
            s["ws"] = _scratch(binding.values_workspace_bytes(n, N, S))
    s["case"] = case
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "eval":
        o = binding.split_eval_device(s["tour"], s["lens"], s["dist"], s["dem"], case["Q"], max_len=case["n"],
                                      out=s["out"], workspace=s["ws"])
        return {"costs": o.costs, "sums": o.sums, "means": o.means}
    if kind == "batch":
        o = s["plan"].launch()
        return {"costs": o.costs, "sums": o.sums, "means": o.means}
    if kind == "routes":
        o = binding.split_routes_device(s["tour"], s["dist"], s["dem"], case["Q"], out=s["out"], workspace=s["ws"])
        return {"costs": o.costs, "pred": o.pred, "cuts": o.cuts, "nroutes": o.nroutes}
    if kind == "variant":
        o = binding.split_variant_device(s["tour"], s["dist"], s["dem"], case["Q"], beta=case["beta"], K=case["K"],
                                         out=s["out"], workspace=s["ws"])
        return {"costs": o.costs, "status": o.status}
    if kind == "values":
        V, st = binding.split_values_device(s["tour"], s["dist"], s["dem"], case["Q"], V=s["out"][0],
                                            status=s["out"][1], workspace=s["ws"])
        return {"V": V, "status": st}
    if case["U"] <= 31:
        JT, arg = binding.ou_dp(case["U"], s["demand"], s["cost"], s["cap"], s["h"], s["u"], s["rho"], s["J0"],
                                out=s["out"])
    else:
        A = binding.ou_transitions(case["U"], s["demand"], s["cost"], s["cap"], s["h"], s["u"], s["rho"], out=s["A"])
        JT, arg = binding.minplus_forward(A, s["J0"], shared=False)
    return {"JT": JT, "arg": arg, "path": binding.minplus_backtrack(JT, arg)}


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
def work(case):
    """Inputs read once and outputs written once; one operation per admissible
    (scenario, predecessor, position), from the mean route length."""
    kind = case["kind"]
    if kind == "inventory":
        B, T, R, m = case["customers"] * case["scenarios"], case["T"], case["R"], case["U"] + 1
        # demands, options, J_0 in; J_T, minimisers, paths out; two sources
        # per level and one look at every option
        return {"bytes": 4.0 * B * (T + 2 * T * R + 2 * m + T * m + T + 1), "flops": float(B) * T * (3 * m + R)}
    if kind == "batch":
        T, N, S = case["T"], case["n_hi"], case["S"]
        n, mean = (case["n_lo"] + case["n_hi"]) / 2, 8.5
        return {"bytes": 2.0 * S * N + 4.0 * T * S + 4.0 * (N + 1) ** 2 + 4.0 * T * n + 16.0 * T,
                "flops": float(T) * S * n * min(n, case["Q"] / mean)}
    n, N, S = case["n"], case["N"], case["S"]
    mean = (case["mu_hi"] + 1) / 2
    stops = min(n / 2, case["Q"] / mean)
    byts = 2.0 * S * N + 4.0 * S + 4.0 * (N + 1) ** 2 + 4.0 * n
    ops = float(S) * n * stops
    if kind == "routes":
        byts += 2.0 * S * n + 2.0 * S * n / max(1.0, 0.7 * stops) + 4.0 * S
    elif kind == "values":
        byts += 4.0 * S * n
    elif kind == "variant" and case["beta"] >= 0:
        ops += 2.0 * S * n  # the overloaded predecessors fold into one minimum
    return {"bytes": byts, "flops": ops}


# ---------------------------------------------------------------------------
# the definitions, in 64-bit integers
# ---------------------------------------------------------------------------
def _route_costs(tour, dist):
    """W[p, i]: cost of the route over tour positions p+1..i (int64 [n, n+1])."""
    c = tour.astype(np.int64)
    n = c.size
    d = dist.astype(np.int64)
    arcs = np.concatenate([[0], np.cumsum(d[c[:-1], c[1:]])]) if n > 1 else np.zeros(1, np.int64)
    out = np.full((n, n + 1), BIG, np.int64)
    for p in range(n):
        out[p, p + 1:] = d[0, c[p]] + (arcs[p:] - arcs[p]) + d[c[p:], 0]
    return torch.from_numpy(out).to(DEV)


def _split(tour, dist, dem, Q, beta=-1, prev=None, pred=None):
    """V [n+1, S]; with `prev`, one more route than `prev`'s values; `pred`
    receives the smallest minimising predecessors."""
    n, S = tour.size, dem.shape[0]
    Wc = _route_costs(tour, dist)
    idx = torch.from_numpy(tour.astype(np.int64) - 1).to(DEV)
    load = torch.zeros((n + 1, S), dtype=torch.int64, device=DEV)
    for j in range(n):
        load[j + 1] = load[j] + dem[:, idx[j]]
    V = torch.full((n + 1, S), BIG, dtype=torch.int64, device=DEV)
    V[0] = 0 if prev is None else BIG
    src = V if prev is None else prev
    order = torch.arange(n, device=DEV)[:, None]
    for j in range(1, n + 1):
        p0 = 0
        if beta < 0:  # no scenario's route ending here starts before p0
            p0 = int((load[j] - load[:j] <= Q).any(dim=1).to(torch.int8).argmax())
        cand = src[p0:j] + Wc[p0:j, j][:, None]
        over = (load[j] - load[p0:j]) - Q
        cand = torch.where(over > 0, BIG, cand) if beta < 0 else cand + beta * over.clamp_(min=0)
        V[j] = cand.amin(dim=0).clamp_(max=BIG)
        if pred is not None:
            best = torch.where(cand == V[j], order[p0:j], BIG).amin(dim=0)
            pred[j - 1] = torch.where(V[j] >= BIG, 0xFFFF, best)
    return V


def _costs(v):
    return torch.where(v >= BIG, INF, v)


def _sum_mean(costs):
    if int((costs == INF).any()):
        return float("inf"), (1 << 63) - 1
    total = int(costs.sum())
    return total / costs.numel(), total


def exact(case, seed):
    kind = case["kind"]
    if kind == "inventory":
        return None  # whole numbers throughout
    if kind == "batch":
        s = _batch_inputs(case, seed)
        dist, tours = s["dist"].cpu().numpy(), s["tours"].cpu().numpy()
        costs, sums, means, off = [], [], [], 0
        for k in s["lens"].cpu().tolist():
            costs.append(_costs(_split(tours[off:off + k], dist, s["dem"], case["Q"])[-1]))
            off += k
            mean, total = _sum_mean(costs[-1])
            sums.append(total)
            means.append(mean)
        return {"costs": torch.stack(costs), "sums": torch.tensor(sums), "means": torch.tensor(means, dtype=torch.float64)}
    s = _tour_inputs(case, seed)
    tour, dist = s["tour"].cpu().numpy(), s["dist"].cpu().numpy()
    if kind == "eval":
        costs = _costs(_split(tour, dist, s["dem"], case["Q"])[-1])
        mean, total = _sum_mean(costs)
        return {"costs": costs[None], "sums": torch.tensor([total]), "means": torch.tensor([mean], dtype=torch.float64)}
    if kind == "values":
        return {"V": _costs(_split(tour, dist, s["dem"], case["Q"])[1:]), "status": torch.zeros(1, dtype=torch.int64)}
    if kind == "routes":
        pred = torch.empty((case["n"], case["S"]), dtype=torch.int64, device=DEV)
        V = _split(tour, dist, s["dem"], case["Q"], pred=pred)
        signed = torch.where(pred > 32767, pred - 65536, pred)  # the outputs are 16-bit words held as int16
        return {"costs": _costs(V[-1]), "pred": signed, "cuts": None, "nroutes": None}
    if case["K"] and case["K"] * case["n"] ** 2 * case["S"] > 5e11:
        return None  # a pass over every pair for each vehicle: too long here
    if not case["K"]:
        best = _split(tour, dist, s["dem"], case["Q"], beta=case["beta"])[-1]
    else:
        J = torch.full((case["n"] + 1, case["S"]), BIG, dtype=torch.int64, device=DEV)
        J[0] = 0
        best = torch.full((case["S"],), BIG, dtype=torch.int64, device=DEV)
        for _ in range(min(case["K"], case["n"])):
            J = _split(tour, dist, s["dem"], case["Q"], beta=case["beta"], prev=J)
            best = torch.minimum(best, J[-1])
    return {"costs": _costs(best), "status": torch.zeros(1, dtype=torch.int64)}
