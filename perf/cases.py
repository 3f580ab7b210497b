"""The work a user of this library has it do, as cases that can be timed and compared.

A case names a call (or the calls of one turn of a serving loop), the shape of the variant table and the
number of queries; everything else follows from a seed.  The distributions are those of ``workloads/``
(accuracies over tens of percent, latencies over three decades, hardware prices over one, Zipf or uniform
popularity of the tasks), drawn on the device where they are large.

calls
  select      the plain selection on a loaded table
  closest     the same, with the closest variant for the queries that nothing satisfies
  stream      a load report on a tenth of the variants, then the selection (a turn of the serving loop)
  tiered      a state report on a twentieth of the variants, then the state-aware selection
  cluster     a report on workers and running instances (loads and states), then the selection with workers
  case1       variant, tier, worker and closest variant of every query in one call
  scale       scaling decisions on a rise in load;  scale_down: the regular check the other way
tables
  even        the same number of variants for every task
  skewed      lognormal numbers of variants (sigma 1.5) around the stated mean
  pareto      dearer variants are more accurate and faster throughout, so that any of them can be the answer
"""
import math

import numpy as np
import torch

import paper_1905_13348_amd as infaas

BATCH_SIZES = (1, 2, 4, 8, 16, 32, 64, 128)
SCALE_CALLS = ("scale", "scale_down")


def _case(call, table, tasks, mean, batches, queries, popularity="uniform", slo="unimodal"):
    return {"call": call, "table": table, "tasks": tasks, "mean": mean, "batches": batches, "queries": queries,
            "popularity": popularity, "slo": slo}


def listed():
    cases = {
        # a small deployment that decides every few milliseconds' arrivals: launches and host work count
        "select_tiny": _case("select", "even", 8, 32, 4, 10_000),
        # an ordinary registry and batch
        "select_medium": _case("select", "even", 100, 200, 8, 1_000_000),
        # the library's main workload: thousands of variants per task, popular tasks first
        "select_thousands": _case("select", "even", 50, 2000, 8, 16_000_000, "zipf"),
        # many tasks of very different sizes, the largest batch
        "select_skewed": _case("select", "skewed", 1000, 100, 8, 64_000_000, "uniform", "bimodal"),
        # the same registry asked for a modest, ragged batch
        "select_skewed_ragged": _case("select", "skewed", 1000, 100, 8, 200_003, "uniform", "bimodal"),
        # a registry without dominated variants, which no index can thin out
        "select_pareto": _case("select", "pareto", 50, 2000, 8, 1_000_003, "zipf"),
        # one turn of the serving loop under changing load
        "stream_thousands": _case("stream", "even", 50, 2000, 8, 4_000_000, "zipf"),
        # suggestions for queries that cannot be met, at a ragged size
        "closest_ragged": _case("closest", "even", 50, 2000, 8, 5_000_011, "zipf"),
        # one turn of the loop with workers and instance states, an ordinary cluster
        "cluster_medium": _case("cluster", "even", 100, 200, 8, 1_000_000),
        # everything the selection can say about a query, at the main workload's size
        "case1_thousands": _case("case1", "even", 50, 2000, 8, 16_000_000, "zipf"),
        # autoscaling decisions for many running variants at once, both directions
        "scale_thousands": _case("scale", "even", 50, 2000, 8, 4_000_000),
        "scale_down_ragged": _case("scale_down", "even", 100, 200, 8, 700_001),
    }
    return [dict(c, name=name) for name, c in cases.items()]


def draw(rng):
    def spread(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    call = rng.choice(("select", "select", "select", "closest", "stream", "tiered", "cluster", "case1", "scale", "scale_down"))
    table = "even" if call not in ("select", "stream", "closest") else rng.choice(("even", "even", "skewed", "pareto"))
    if table == "skewed":
        tasks, mean = spread(100, 1000), spread(30, 100)
    else:
        tasks = spread(8, 200)
        mean = spread(32, min(2000, 100_000 // tasks))
    most = {"select": 64_000_000, "closest": 16_000_000, "stream": 8_000_000, "case1": 16_000_000}.get(call, 4_000_000)
    if table == "pareto":   # every variant may have to be looked at
        most = min(most, (100_000_000 if call == "closest" else 2_000_000_000) // mean, 8_000_000)
    return _case(call, table, tasks, mean, rng.choice((1, 3, 4, 8)), spread(1000, most) | 1,
                 rng.choice(("uniform", "zipf")), rng.choice(("unimodal", "bimodal")))


# ---------------------------------------------------------------- inputs

def _sizes(case, rng):
    T, mean = case["tasks"], case["mean"]
    if case["table"] != "skewed":
        return np.full(T, mean, dtype=np.int64)
    n = np.rint(rng.lognormal(math.log(mean) - 1.125, 1.5, size=T)).astype(np.int64)
    return np.clip(n, 1, 20_000)


def _table(case, rng):
    """Host columns of the variant table, rows shuffled."""
    sizes = _sizes(case, rng)
    T, B, V = case["tasks"], case["batches"], int(sizes.sum())
    task = np.repeat(np.arange(T), sizes)
    nth = np.arange(V) - np.repeat(np.cumsum(sizes) - sizes, sizes)   # number of the variant within its task
    of = np.repeat(sizes, sizes)
    b = np.asarray(BATCH_SIZES[:B], dtype=np.int64)[None, :]
    if case["table"] == "pareto":
        acc = 5000 + 4500 * nth // of
        lat = (60_000 - 59_000 * nth // of)[:, None] + 10 * np.arange(B)[None, :]
        cost = (100 + nth)[:, None] + np.arange(B)[None, :]
        queue = np.zeros(V, dtype=np.int64)
    else:
        acc = rng.integers(5000, 9501, size=V)
        price = np.array([1, 4, 9])[rng.integers(0, 3, size=V)]
        base = np.clip(rng.lognormal(math.log(2000.0), 1.0, size=V), 100.0, 500_000.0)
        lat = np.maximum(np.rint(base[:, None] * b.astype(np.float64) ** rng.uniform(0.3, 1.0, size=V)[:, None]), 1).astype(np.int64)
        cost = (lat * price[:, None] + b - 1) // b
        queue = rng.integers(0, 50_001, size=V)
    p = rng.permutation(V)
    return {"task": task[p].astype(np.int32), "acc": acc[p].astype(np.int32), "lat": lat[p].astype(np.int32),
            "cost": cost[p].astype(np.int32), "queue": queue[p].astype(np.int32)}


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _slo(case, n, g):
    def logn(median):
        return torch.exp(torch.randn(n, generator=g, device="cuda") + math.log(median))
    if case["slo"] == "unimodal":
        s = logn(20_000.0)
    else:
        s = torch.where(torch.rand(n, generator=g, device="cuda") < 0.5, logn(5000.0), logn(200_000.0))
    return s.round().clamp(1000, 2_000_000).to(torch.int32)


def _uniform(lo, hi, n, g):   # lo .. hi inclusive
    return torch.randint(lo, hi + 1, (n,), generator=g, device="cuda", dtype=torch.int32)


def _queries(case, seed):
    g, n, T = _gen(seed), case["queries"], case["tasks"]
    if case["popularity"] == "uniform":
        task = _uniform(0, T - 1, n, g)
    else:
        w = torch.arange(1, T + 1, device="cuda", dtype=torch.float64) ** -1.1
        u = torch.rand(n, generator=g, device="cuda")
        task = torch.searchsorted((torch.cumsum(w, 0) / w.sum()).to(torch.float32), u).clamp(max=T - 1).to(torch.int32)
    return [task, _slo(case, n, g), _uniform(5000, 9500, n, g), _uniform(0, case["batches"] - 1, n, g)]


def _load_report(case, V, rng):
    rows = rng.choice(V, size=max(1, V // 10), replace=False).astype(np.int32)
    return rows, rng.integers(0, 200_001, size=rows.size).astype(np.int32)


def _states(V, rng):
    return (rng.choice(4, size=V, p=(0.50, 0.40, 0.05, 0.05)).astype(np.int32),
            np.clip(np.rint(rng.lognormal(math.log(20_000.0), 1.5, size=V)), 100, 5_000_000).astype(np.int32))


def _cluster(V, state, rng):
    """Workers of three kinds of hardware; every loaded variant runs 1 + Poisson(1) instances, at most 8, on
    distinct workers of its kind."""
    W = 3 * max(16, min(341, V // 80))
    worker_hw = rng.permutation(np.arange(W) % 3).astype(np.int32)
    by_class = np.argsort(worker_hw, kind="stable").reshape(3, -1)
    variant_hw = rng.integers(0, 3, size=V).astype(np.int32)
    count = np.where(state != 0, np.minimum(1 + rng.poisson(1.0, size=V), 8), 0)
    inst_variant = np.repeat(np.arange(V), count)
    nth = np.arange(inst_variant.size) - np.repeat(np.cumsum(count) - count, count)
    first = rng.integers(0, W // 3, size=V)
    inst_worker = by_class[variant_hw[inst_variant], (first[inst_variant] + nth) % (W // 3)]
    p = rng.permutation(inst_variant.size)
    return {"worker_hw": worker_hw, "worker_util": rng.integers(0, 10_001, size=W).astype(np.int32), "variant_hw": variant_hw,
            "inst_variant": inst_variant[p].astype(np.int32), "inst_worker": inst_worker[p].astype(np.int32),
            "inst_load": rng.integers(0, 1001, size=p.size).astype(np.int32)}


def _instance_states(n, rng):
    return rng.choice(np.array([1, 2, 3], dtype=np.int32), size=n, p=(0.80, 0.12, 0.08)).astype(np.int32)


def _report(n, share, rng):
    return rng.choice(n, size=max(1, int(n * share)), replace=False).astype(np.int32)


def _scaling(t, case, rng):
    """About a dozen variants of a task share an architecture."""
    sizes = np.bincount(t["task"], minlength=case["tasks"])
    archs = np.maximum(1, np.rint(sizes / 12.0).astype(np.int64))
    first = np.cumsum(archs) - archs
    V = t["task"].size
    arch = first[t["task"]] + np.floor(rng.random(V) * archs[t["task"]]).astype(np.int64)
    return (arch.astype(np.int32), np.clip(np.rint(rng.lognormal(math.log(200.0), 1.2, size=V)), 1, 200_000).astype(np.int32),
            rng.integers(50, 2001, size=V).astype(np.int32),
            np.clip(np.rint(rng.lognormal(math.log(20_000.0), 1.5, size=V)), 100, 5_000_000).astype(np.int32))


def _requests(case, qps, seed, rng):
    g, n, down = _gen(seed), case["queries"], case["call"] == "scale_down"
    variant = _uniform(0, qps.size - 1, n, g)
    inst = 1 + torch.poisson(torch.full((n,), 2.0 if down else 1.0, device="cuda"), generator=g).to(torch.int32)
    lo, hi = (0.0, 1.2) if down else (0.5, 4.0)
    u = lo + (hi - lo) * torch.rand(n, generator=g, device="cuda", dtype=torch.float64)
    load = (_dev(qps)[variant.long()].double() * inst * u).round().clamp(max=1e9).to(torch.int32)
    return [variant, inst, load, _slo(case, n, g), _uniform(0, case["batches"] - 1, n, g)]


def _dev(a):
    return torch.from_numpy(a).cuda()


def _outputs(case, k):
    return [torch.empty(case["queries"], dtype=torch.int32, device="cuda") for _ in range(k)]


def prepare(case, seed):
    """A handle with its table (and states, cluster or scaling profile), the queries on the device, the result
    arrays, and the report that a turn of a loop begins with."""
    call, rng = case["call"], np.random.default_rng([seed, 1])
    t = _table(case, rng)
    V = t["task"].size
    h = infaas.Selector(case["tasks"], BATCH_SIZES[:case["batches"]], device=torch.cuda.current_device())
    h.load_variants(t["task"], t["acc"], t["lat"], t["cost"], t["queue"])
    s = {"call": call, "handle": h}
    if call in SCALE_CALLS:
        profile = _scaling(t, case, rng)
        h.load_scaling(*profile, lambda_per_s=50, slack_pct=105)
        s["in"], s["out"] = _requests(case, profile[1], seed, rng), _outputs(case, 3)
        return s
    s["in"] = _queries(case, seed)
    s["out"] = _outputs(case, {"closest": 2, "tiered": 2, "cluster": 3, "case1": 4}.get(call, 1))
    if call == "stream":
        s["report"] = [_dev(a) for a in _load_report(case, V, rng)]
    if call in ("tiered", "cluster", "case1"):
        state, load_us = _states(V, rng)
        h.load_states(state, load_us)
        if call == "tiered":
            s["report"] = [_dev(_report(V, 0.05, rng)), _dev(rng.choice(4, size=max(1, int(V * 0.05)), p=(0.50, 0.40, 0.05, 0.05)).astype(np.int32))]
        else:
            c = _cluster(V, state, rng)
            h.load_workers(**c)
            if call == "cluster":
                W, n = c["worker_hw"].size, c["inst_variant"].size
                h.load_instance_states(_instance_states(n, rng))
                w, i, k = _report(W, 0.10, rng), _report(n, 0.10, rng), _report(n, 0.05, rng)
                s["report"] = [_dev(w), _dev(rng.integers(0, 10_001, size=w.size).astype(np.int32)),
                               _dev(i), _dev(rng.integers(0, 1001, size=i.size).astype(np.int32))]
                s["states"] = [_dev(k), _dev(_instance_states(k.size, rng))]
    h.reserve(case["queries"])
    return s


# ---------------------------------------------------------------- one pass

def run(s):
    h, call = s["handle"], s["call"]
    if call == "select":
        h.select(*s["in"], *s["out"])
    elif call == "closest":
        h.select_closest(*s["in"], *s["out"])
    elif call == "stream":
        h.update_load(*s["report"])
        h.select(*s["in"], *s["out"])
    elif call == "tiered":
        h.update_state(*s["report"])
        h.select_tiered(*s["in"], *s["out"])
    elif call == "cluster":
        h.update_workers(*s["report"])
        h.update_instance_states(*s["states"])
        h.select_workers(*s["in"], *s["out"])
    elif call == "case1":
        h.select_workers_closest(*s["in"], *s["out"])
    elif call == "scale":
        h.scale(*s["in"], *s["out"])
    else:
        h.scale_down(*s["in"], *s["out"])
    return s["out"]


def work(case):
    """The query fields read once, the results written once, the variant table (accuracy, queue, row; latency and
    cost per batch size) read once; for scaling decisions the profile (architecture, throughput, cost, loading
    latency; latency per batch size); reports as (index, value) pairs."""
    call, V, B, n = case["call"], case["tasks"] * case["mean"], case["batches"], case["queries"]
    if call in SCALE_CALLS:
        return {"bytes": 32 * n + V * (16 + 4 * B), "flops": 0}
    outputs = {"closest": 2, "tiered": 2, "cluster": 3, "case1": 4}.get(call, 1)
    size = (16 + 4 * outputs) * n + V * (12 + 8 * B)
    size += {"stream": 8 * V // 10, "tiered": 8 * V // 20, "cluster": 2 * V}.get(call, 0)
    return {"bytes": size, "flops": 0}


def tolerance(case):
    """Rows, tiers, workers and actions: whole numbers, the same for every correct implementation."""
    return "exact"


def exact(case, seed):
    """The plain selection by brute force over every query's slice; None for the other calls (their results are
    whole numbers too)."""
    if case["call"] not in ("select", "stream"):
        return None
    rng = np.random.default_rng([seed, 1])
    t = _table(case, rng)
    V, B, n = t["task"].size, case["batches"], case["queries"]
    queue = t["queue"].astype(np.int64)
    if case["call"] == "stream":
        rows, values = _load_report(case, V, rng)
        queue[rows] = values
    task, slo, acc, batch = _queries(case, seed)
    slices = task.long() * B + batch
    order = torch.argsort(slices, stable=True)
    at = np.concatenate([[0], torch.cumsum(torch.bincount(slices, minlength=case["tasks"] * B), 0).cpu().numpy()])
    out = torch.full((n,), -1, dtype=torch.int64, device="cuda")
    by_task = np.argsort(t["task"], kind="stable")
    ends = np.concatenate([[0], np.cumsum(np.bincount(t["task"], minlength=case["tasks"]))])
    for k in range(case["tasks"]):
        rows = by_task[ends[k]:ends[k + 1]]
        for b in range(B):
            r = rows[np.lexsort((rows, t["lat"][rows, b], t["cost"][rows, b]))]   # the order answers are preferred in
            a, l = _dev(t["acc"][r].astype(np.int64)), _dev(t["lat"][r, b].astype(np.int64) + queue[r])
            r = torch.cat([_dev(r.astype(np.int64)), torch.full((1,), -1, device="cuda")])
            place = torch.arange(a.numel(), device="cuda")
            step = max(1, (1 << 26) // a.numel())
            for lo in range(int(at[k * B + b]), int(at[k * B + b + 1]), step):
                q = order[lo:min(lo + step, int(at[k * B + b + 1]))]
                fits = (a[None, :] >= acc[q].long()[:, None]) & (l[None, :] <= slo[q].long()[:, None])
                out[q] = r[torch.where(fits, place[None, :], a.numel()).amin(1)]
    return [out.to(torch.int32)]
