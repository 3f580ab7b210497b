"""Batches small enough to be answered straight from global memory, one lane per query, and batches on both
sides of the size where the LDS mirror (or a tile of queries at a time) takes over: an index that fits the
mirror, one that does so in part, one laid out in groups and one whose headers leave no room for a mirror;
arrays that start 4 bytes into their allocations.  Every answer against the CPU oracle."""
import numpy as np
import pytest

import workloads
from gpu_util import (MEMORY, MIRROR, TILES, Repeated, gpu_select, gpu_select_closest, make_selector, query_args,
                      table_args)
from test_gpu_case1 import gpu_case1
from test_gpu_getvariant import gpu_get_variant
from test_gpu_parity import (_assert_equal_everywhere, _random_queries, _random_table, _staircase_queries,
                             _staircase_table, _table)
from test_gpu_tiered import gpu_select_tiered
from test_gpu_workers import _random_cluster, gpu_select_workers, load_cluster

pytestmark = pytest.mark.gpu


def _many_tasks():
    rng = np.random.default_rng(5)
    return _random_table(rng, 12_000, rng.integers(0, 12, 12_000), 1)


TABLES = {"mirrored": lambda: workloads.make_table(2), "partly": lambda: workloads.make_table(1),
          "groups": lambda: workloads.make_table(3), "no_mirror": _many_tasks}


@pytest.mark.parametrize("kind", list(TABLES))
def test_small_batches(oracle_lib, kind):
    import torch
    tb = TABLES[kind]()
    most = 100_001
    q = workloads.make_queries(1, n=most, seed=77)
    rng = np.random.default_rng(6)
    task, bidx = rng.integers(-1, tb.num_tasks + 1, most).astype(np.int32), rng.integers(-1, tb.B + 1, most).astype(np.int32)
    _, slo, acc, _ = (x.copy() for x in query_args(q))
    slo[::97] = rng.choice([-1, 0, 2**31 - 1, -2**31], slo[::97].size)
    acc[::89] = rng.choice([-2**31, 2**31 - 1], acc[::89].size)
    want = oracle_lib.select(*table_args(tb), task, slo, acc, bidx)
    sel = make_selector(tb, engine=0)
    for shift in (0, 1):
        dev = [torch.cat([torch.zeros(shift, dtype=torch.int32), torch.from_numpy(x)]).cuda()[shift:] for x in (task, slo, acc, bidx)]
        for n in (1, 63, 64, 65, 255, 256, 257, 5003, most - 1, most):
            for call in (sel.select, sel.select_noalloc):
                out = torch.full((n + shift + 3,), -7, dtype=torch.int32, device="cuda")[shift:]
                call(*dev, out, n=n)
                torch.cuda.synchronize()
                got = out.cpu().numpy()
                _assert_equal_everywhere(got[:n], want[:n], f"{kind} N={n} shift={shift} {call.__name__}")
                assert (got[n:] == -7).all()
    info = sel.info()
    assert info["lookup_parked"] >= info["lookup_second_body"] + info["lookup_unanswered"]
    sel.destroy()


def _few_groups():
    rng = np.random.default_rng(15)
    return _random_table(rng, 200, np.full(200, 500), 8)


@pytest.mark.parametrize("kind", list(TABLES) + ["few_groups"])
def test_both_sides_of_the_limit(oracle_lib, kind):
    """As many queries as go a lane per query, and one more, which go through the mirror where it holds the whole index and a tile
    at a time elsewhere.  The statistics are those of what was done: straight from memory every query counts as set aside."""
    tb = _few_groups() if kind == "few_groups" else TABLES[kind]()
    q = workloads.make_queries(1, n=60_001, seed=78)
    rng = np.random.default_rng(7)
    task, bidx = rng.integers(0, tb.num_tasks, q.N).astype(np.int32), rng.integers(0, tb.B, q.N).astype(np.int32)
    qs = (task, *query_args(q)[1:3], bidx)
    sel = make_selector(tb, engine=0)
    assert (sel.info()["index_groups"] > 1) == (kind in ("groups", "few_groups", "no_mirror"))
    assert sel.info()["lookup_route"] == 0
    many = Repeated(sel, sel.select, qs, [oracle_lib.select(*table_args(tb), *qs)])
    limit = many.last_from_memory(2_000_001)
    many.check(limit, MEMORY, kind)
    info = sel.info()
    assert info["lookup_parked"] == limit and info["lookup_global_body"] > limit // 4
    many.check(limit + 1, MIRROR if kind == "mirrored" else TILES, kind)
    assert sel.info()["lookup_parked"] < limit // 2
    sel.destroy()


@pytest.mark.parametrize("kind", ["ties", "staircase62", "staircase63", "staircase300", "one_tier", "masked", "partly", "few_incomplete"])
def test_every_mode_below_and_above_the_limit(oracle_lib, kind):
    """The calls on tables that make their paths differ: ties, two bodies to a slice, slices with more steps than the index keeps
    (all, or so few that the mirror still pays), slices without a variant of one tier or of both, bodies that the mirror does not
    hold.  3001 queries in one call (straight from memory) and the same queries over and over, in a call of 300,100 and, unless
    all slices are incomplete (which goes straight from memory at every size), in one that goes through the LDS mirrors and, with
    states, the lists between the tiers; aligned arrays and others; every element against the CPU oracle."""
    rng = np.random.default_rng(len(kind) * 31)
    if kind == "partly":
        tb, span = _random_table(rng, 100, np.full(100, 190), 8), None
        q = _random_queries(rng, 100, 8, 3001)
    elif kind == "few_incomplete":     # one slice of 1500, most of whose steps the index does not keep
        small, long_ = _random_table(rng, 1499, np.full(1499, 4), 1), _staircase_table(1, 300, B=1)
        tb, span = _table(1500, [1], np.concatenate([small.task_id, long_.task_id + 1499]), np.concatenate([small.acc_bp, long_.acc_bp]),
                          np.concatenate([small.lat_us, long_.lat_us]), np.concatenate([small.cost, long_.cost]),
                          np.concatenate([small.queue_us, long_.queue_us])), None
        q = tuple(np.concatenate(x) for x in zip(_random_queries(rng, 1499, 1, 2000),
                                                 [a + (1499 if k == 0 else 0) for k, a in enumerate(_staircase_queries(rng, long_, 1001, 300))]))
        q = tuple(x.astype(np.int32) for x in q)
    elif kind.startswith("staircase"):
        steps = int(kind[9:])
        tb, span = _staircase_table(5, steps), None
        q = _staircase_queries(rng, tb, 3001, steps)
    else:
        span = 4 if kind == "ties" else None
        tb = _random_table(rng, 9, np.asarray([40, 0, 7, 130, 1, 64, 33, 90, 300]), 3, span=span)
        q = _random_queries(rng, 9, 3, 3001, span=span)
    vals = span if span else 50_000
    state = rng.integers(0, 4, tb.V).astype(np.int32)
    if kind == "one_tier":     # some tasks all Active, some all Inactive
        state = (tb.task_id % 2).astype(np.int32)
    if kind == "masked":       # some tasks that nothing of may be selected from
        state[tb.task_id % 3 == 0] = 2
    load = rng.integers(0, vals, tb.V).astype(np.int32)
    cl = _random_cluster(rng, tb.V, state, vals)
    times = 100
    many = tuple(np.tile(x, times) for x in q)

    def check(got, want, label):
        for g, w, what in zip(got, want, ("variant", "second", "third", "fourth")):
            _assert_equal_everywhere(g, np.tile(w, times) if g.size > w.size else w, f"{kind} {label} {what}")

    def through_the_mirror(call, want, label):
        if kind in ("staircase63", "staircase300"):
            return
        many = Repeated(sel, call, q, want)
        n = many.least_beyond(351_007, 40_000_000, MIRROR)
        for m, shift in ((n, 0), (n + 2, 1)):
            many.check(m, MIRROR, f"{kind} {label}", shift)

    sel = make_selector(tb, engine=2)
    want = oracle_lib.select_closest(*table_args(tb), *q)
    through_the_mirror(sel.select, want[:1], "select")
    for qs in (q, many):
        check(gpu_select_closest(sel, *qs), want, f"closest N={len(qs[0])}")
    through_the_mirror(sel.select_closest, want, "closest")
    if kind == "partly":
        assert sel.info()["lookup_global_body"] > 0
    if kind == "few_incomplete":
        assert sel.info()["lookup_scanned"] > 0
    sel.load_states(state, load)
    load_cluster(sel, cl)
    for name, call, method, want in (
            ("tiered", gpu_select_tiered, sel.select_tiered, oracle_lib.select_tiered(*table_args(tb), state, load, *q)),
            ("case1", gpu_case1, sel.select_tiered_closest, oracle_lib.select_case1(*table_args(tb), state, load, *q)),
            ("workers", gpu_select_workers, sel.select_workers, oracle_lib.select_workers(*table_args(tb), state, load, *cl, *q)),
            ("getvariant", gpu_get_variant, sel.select_workers_closest, oracle_lib.get_variant(*table_args(tb), state, load, *cl, *q))):
        for qs in (q, many):
            check(call(sel, *qs), want, f"{name} N={len(qs[0])}")
        through_the_mirror(method, want, name)
    sel.destroy()


def test_a_small_call_leaves_the_scratch_of_its_size(oracle_lib):
    """One eager call is warm-up enough for a capture of the same size, whichever way a report turns it: after
    a small call the lists between the tiers are there, and nothing is left for infaas_sel_reserve to do."""
    rng = np.random.default_rng(3)
    tb = _random_table(rng, 9, np.full(9, 40), 3)
    q = _random_queries(rng, 9, 3, 5003)
    state, load = rng.integers(0, 4, tb.V).astype(np.int32), rng.integers(0, 50_000, tb.V).astype(np.int32)
    sel = make_selector(tb, engine=0)
    sel.load_states(state, load)
    before = sel.info()["scratch_bytes"]
    for call, want, size in ((gpu_select_tiered, oracle_lib.select_tiered, 16), (gpu_case1, oracle_lib.select_case1, 32)):
        for g, w in zip(call(sel, *q), want(*table_args(tb), state, load, *q)):
            _assert_equal_everywhere(g, w, call.__name__)
        after = sel.info()["scratch_bytes"]
        assert after >= before + size * len(q[0])
        sel.reserve(len(q[0]))
        assert sel.info()["scratch_bytes"] == after
    sel.destroy()


def test_suggestions_around_their_own_limit(oracle_lib):
    """An index that the mirror holds nearly completely and that has second bodies: suggestions turn to the lookup
    kernel earlier than the plain selection."""
    tb = workloads.make_table(2)
    sel = make_selector(tb, engine=0)
    assert sel.info()["index_max_steps"] > 31
    q = query_args(workloads.make_queries(2, n=75_001, seed=9))
    want = oracle_lib.select_closest(*table_args(tb), *q)
    assert (q[1] >= 0).all()
    many = Repeated(sel, sel.select_closest, q, want)
    limit = many.last_from_memory(1_000_001)
    many.check(limit, MEMORY, "closest")
    assert sel.info()["lookup_parked"] == limit
    many.check(limit + 1, MIRROR, "closest")
    assert 0 < sel.info()["lookup_parked"] < limit // 2
    assert Repeated(sel, sel.select, q, want[:1]).last_from_memory(1_000_001) > limit
    sel.destroy()


@pytest.mark.parametrize("n", [3001, 400_001 * 15])
def test_a_call_captured_without_warm_up(oracle_lib, n):
    """A call may be captured before any other: it goes straight from memory, which needs no lists, at a size too that would go
    through the mirrors.  Its replays answer, and the eager call behind them allocates the lists."""
    import torch
    rng = np.random.default_rng(4)
    tb = _random_table(rng, 9, np.full(9, 40), 3)
    state, load = rng.integers(0, 4, tb.V).astype(np.int32), rng.integers(0, 50_000, tb.V).astype(np.int32)
    times = 1 if n < 10_000 else 15
    n //= times
    sets = [_random_queries(rng, 9, 3, n) for _ in range(3)]
    want = [[np.tile(w, times) for w in oracle_lib.select_case1(*table_args(tb), state, load, *q)] for q in sets]
    sets = [[np.tile(x, times) for x in q] for q in sets]
    n *= times
    loaded = make_selector(tb, engine=0)          # (so that the kernel's code is on the device)
    loaded.load_states(state, load)
    gpu_case1(loaded, *sets[0])
    sel = make_selector(tb, engine=0)
    sel.load_states(state, load)
    before = sel.info()["scratch_bytes"]
    dq = [torch.zeros(n, dtype=torch.int32, device="cuda") for _ in range(4)]
    out = [torch.zeros(n, dtype=torch.int32, device="cuda") for _ in range(3)]
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        sel.select_tiered_closest(*dq, *out)
    assert sel.info()["scratch_bytes"] == before and sel.info()["lookup_route"] == MEMORY
    for rnd in range(4):
        for d, x in zip(dq, sets[rnd % 3]):
            d.copy_(torch.from_numpy(x))
        for o in out:
            o.fill_(-9)
        graph.replay()
        torch.cuda.synchronize()
        for g, w in zip(out, want[rnd % 3]):
            _assert_equal_everywhere(g.cpu().numpy(), w, f"replay {rnd}")
    sel.select_tiered_closest(*dq, *out)
    torch.cuda.synchronize()
    assert sel.info()["scratch_bytes"] >= before + 32 * n
    assert sel.info()["lookup_route"] == (MEMORY if n < 10_000 else MIRROR)
    for g, w in zip(out, want[rnd % 3]):
        _assert_equal_everywhere(g.cpu().numpy(), w, "eager")
    loaded.destroy()
    sel.destroy()


def _pool_bytes(sel):
    """Bytes of the bodies of the handle's index (of the Active tier, if it has states), as of its latest selection."""
    i = sel.info()
    return i["index_bytes"] - 16 * i["num_slices"] - 4 * (i["index_steps"] + 1)


LENGTHS = [1, 6, 7, 8, 9, 15, 16, 17, 23, 24, 25, 30, 31, 32, 38, 39, 61, 62, 63]


@pytest.mark.parametrize("steps", LENGTHS)
def test_bodies_of_every_length(oracle_lib, steps):
    """Six slices: bounds that meet each key exactly, miss it by one, meet all or none.  Straight from memory and, where the index holds
    the slices completely, in their bodies in the mirror."""
    tb = _staircase_table(3, steps)
    rows = np.arange(tb.V)
    acc = np.concatenate([tb.acc_bp[rows] + d for d in (-1, 0, 1)] + [np.full(tb.V, x) for x in (-2**31, 2**31 - 1)])
    tot = (tb.lat_us[:, 0] + tb.queue_us).astype(np.int64)
    slo = np.concatenate([tot + d for d in (-1, 0, 1)] + [np.full(tb.V, x) for x in (0, 2**31 - 1)])
    a, s = np.repeat(acc, 5), np.concatenate([np.roll(slo, k) for k in (0, 1, tb.V, 2 * tb.V, 3 * tb.V)])
    n = a.size
    q = tuple(np.clip(x, -2**31, 2**31 - 1).astype(np.int32) for x in
              (np.arange(n) % 3, s, a, np.arange(n) // 3 % tb.B))
    want = oracle_lib.select(*table_args(tb), *q)
    sel = make_selector(tb, engine=2)
    _assert_equal_everywhere(gpu_select(sel, *q), want, f"{steps} steps")
    assert (want >= 0).any() and (want < 0).any()
    if steps <= 62:
        Repeated(sel, sel.select, q, [want]).check(400_001, MIRROR, f"{steps} steps")
        closest = Repeated(sel, sel.select_closest, q, oracle_lib.select_closest(*table_args(tb), *q))
        closest.check(closest.least_beyond(400_001, 2_000_000, MIRROR), MIRROR, f"{steps} steps, closest")
    assert _pool_bytes(sel) <= 24 * 1024
    sel.destroy()


@pytest.mark.parametrize("steps", LENGTHS)
def test_many_bodies_of_every_length(oracle_lib, steps):
    """Staircases that end in front of, at and behind every lane's share of a line, and bounds that meet a key exactly, miss it by one,
    meet all or none, on tables as small as in the test above and on ones whose lines are more than L1 holds.  Batches that give a
    wavefront 16, 32 and 64 queries; every call, half of the tasks in either tier (whose own staircases have as many steps); where
    the index holds the small tables' slices completely, through the mirrors too."""
    rng = np.random.default_rng([71, steps])
    body = sum(14 * ((k + 2) // 2 * 2) for k in (min(steps, 31), min(steps, 62) - 31) if k > 0)
    for half, large in ((2, False), (-(-110_000 // (2 * body)), True)):
        tb = _staircase_table(2 * half, steps)
        nth = np.arange(tb.V) % steps
        load = (200 * nth).astype(np.int32)                      # in the Inactive tier the more accurate, the slower
        state = (np.arange(tb.V) // steps % 2).astype(np.int32)  # odd tasks Active, even ones Inactive
        n = 90_001
        row = rng.integers(0, tb.V, n)
        bidx = rng.integers(0, 2, n)
        key = tb.lat_us[row, bidx].astype(np.int64) + np.where(rng.random(n) < 0.5, load[row], 0)
        other = np.clip(row + rng.integers(-2, 3, n), 0, tb.V - 1)
        acc = tb.acc_bp[other].astype(np.int64) + rng.integers(-1, 2, n)
        slo = key + rng.integers(-1, 2, n)
        acc[::17], slo[::19] = rng.choice([-2**31, 2**31 - 1], acc[::17].size), rng.choice([0, 2**31 - 1], slo[::19].size)
        q = tuple(x.astype(np.int32) for x in (tb.task_id[row], slo, acc, bidx))
        sel = make_selector(tb, engine=2)
        want = oracle_lib.select(*table_args(tb), *q)
        closest = oracle_lib.select_closest(*table_args(tb), *q)
        assert (want >= 0).any() and (want < 0).any()
        for size in (3001, 50_001, 74_001, 90_001):
            cut = tuple(x[:size] for x in q)
            _assert_equal_everywhere(gpu_select(sel, *cut), want[:size], f"{steps} steps N={size}")
            for g, w in zip(gpu_select_closest(sel, *cut), closest):
                _assert_equal_everywhere(g, w[:size], f"{steps} steps closest N={size}")
        assert (_pool_bytes(sel) > 96 * 1024) == large
        sel.load_states(state, load)
        for call, want in ((gpu_select_tiered, oracle_lib.select_tiered(*table_args(tb), state, load, *q)),
                           (gpu_case1, oracle_lib.select_case1(*table_args(tb), state, load, *q))):
            assert all((want[1] == tier).any() for tier in (0, 1, 2))
            for size in (3001, 50_001, 90_001, 180_002):
                many = tuple(np.tile(x, 2)[:size] for x in q)
                for g, w in zip(call(sel, *many), want):
                    _assert_equal_everywhere(g, np.tile(w, 2)[:size], f"{steps} steps {call.__name__} N={size}")
            if not large and steps <= 62:
                method = sel.select_tiered if call is gpu_select_tiered else sel.select_tiered_closest
                Repeated(sel, method, q, want).check(6_000_001, MIRROR, f"{steps} steps {call.__name__}")
        assert (_pool_bytes(sel) > 96 * 1024) == large
        sel.destroy()


@pytest.mark.parametrize("workers", [False, True])
def test_both_sides_of_the_state_aware_limit(oracle_lib, workers):
    """As many queries as one kernel answers for both tiers, and one query more: straight from memory every valid query counts as
    set aside, in both tiers that look at it; the lookup kernels set few aside.  Every element against the CPU oracle."""
    from test_gpu_workers import cluster_args, load_cluster
    tb = workloads.make_table(0)           # both mirrors hold everything
    st = workloads.make_states(0, tb.V)
    q = tuple(x[:5000] for x in query_args(workloads.make_queries(0)))
    sel = make_selector(tb, engine=0)
    sel.load_states(st.state, st.load_us)
    if workers:
        cl = cluster_args(workloads.make_workers(0, st))
        load_cluster(sel, cl)
        want = oracle_lib.select_workers(*table_args(tb), st.state, st.load_us, *cl, *q)
    else:
        want = oracle_lib.select_tiered(*table_args(tb), st.state, st.load_us, *q)
    many = Repeated(sel, sel.select_workers if workers else sel.select_tiered, q, want)
    limit = many.last_from_memory(8_000_001)
    many.check(limit, MEMORY, "two tiers")
    assert sel.info()["lookup_parked"] >= limit
    many.check(limit + 1, MIRROR, "two tiers")
    assert sel.info()["lookup_parked"] < limit // 2
    sel.destroy()
