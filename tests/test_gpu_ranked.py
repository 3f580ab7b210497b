"""Slices the staircase index cannot hold (more steps than it keeps, or accuracies beyond its 16-bit
keys), answered from their entries in rank order through TableView::rank_nodes: slice lengths around
the sizes of a node's entries (16), a level (256, 4096, 65536) and a sorted block (256), tables on which
the first candidate fits, tables on which many do not, every answer against the CPU oracle."""
import numpy as np
import pytest

from gpu_util import gpu_select, make_selector, table_args, to_dev
from test_gpu_case1 import gpu_case1
from test_gpu_parity import _assert_equal_everywhere, _table
from test_gpu_tiered import gpu_select_tiered

pytestmark = pytest.mark.gpu

LENGTHS = (63, 64, 65, 255, 256, 257, 272, 511, 513, 2000, 4095, 4096, 4097, 8449)


def _ranked_table(kind, lengths, B, rng):
    """Tasks of the given lengths; in rank (= cost) order:
    'stairs'  accuracy rises and latency falls, every entry can be the answer
    'mixed'   two such families in turn, one cheap on latency and one on accuracy: a query for both has none
    'noisy'   both random, the cost rising with accuracy and speed and a little at random
    'wide'    as 'noisy', accuracies over the whole of int32: no slice has a body"""
    task, acc, lat, cost = [], [], [], []
    for t, n in enumerate(lengths):
        i = np.arange(n, dtype=np.int64)
        if kind == "stairs":
            a, l, c = 5000 + i, 2_000_000 - 20 * i, 10 + i
        elif kind == "mixed":
            a = np.where(i % 2 == 0, 5000 + i // 4, 40_000 + i // 4)
            l = np.where(i % 2 == 0, 200_000 - 2 * i, 500_000 - 3 * i)
            c = 10 + i
        else:
            x, y = rng.random(n), rng.random(n)
            a = 5000 + 9000 * x
            l, c = 1000 + 250_000 * y, 10 + 20_000 * (x + 1 - y + 0.1 * rng.random(n))
            if kind == "wide":
                a = -2.0**31 + 4294967295.0 * x
        task.append(np.full(n, t)); acc.append(a); lat.append(l); cost.append(c)
    lat, cost = np.concatenate(lat).astype(np.int64)[:, None], np.concatenate(cost).astype(np.int64)[:, None]
    b = np.arange(B, dtype=np.int64)[None, :]
    tb = _table(len(lengths), list(range(1, B + 1)), np.concatenate(task), np.concatenate(acc).astype(np.int64), lat + b, cost + b,
                np.zeros(sum(lengths), np.int64))
    p = rng.permutation(tb.V)
    return _table(tb.num_tasks, tb.batch_sizes, tb.task_id[p], tb.acc_bp[p], tb.lat_us[p], tb.cost[p], tb.queue_us[p])


def _ranked_queries(tb, n, rng):
    """Bounds at, just below and just above the figures of random variants, and values no table has."""
    v, w = rng.integers(0, tb.V, n), rng.integers(0, tb.V, n)
    task, bidx = tb.task_id[v].astype(np.int64), rng.integers(0, tb.B, n)
    same = rng.random(n) < 0.5
    w = np.where(same, v, w)
    acc = tb.acc_bp[v].astype(np.int64) + rng.integers(-1, 2, n)
    slo = tb.lat_us[w, bidx].astype(np.int64) + rng.integers(-1, 2, n)
    odd = rng.random(n)
    task[odd < 0.02] = rng.choice([-1, tb.num_tasks, 2**31 - 1], int((odd < 0.02).sum()))
    bidx[(odd > 0.02) & (odd < 0.04)] = rng.choice([-1, tb.B], int(((odd > 0.02) & (odd < 0.04)).sum()))
    acc[(odd > 0.04) & (odd < 0.08)] = rng.choice([-2**31, 2**31 - 1, 0], int(((odd > 0.04) & (odd < 0.08)).sum()))
    slo[(odd > 0.08) & (odd < 0.12)] = rng.choice([-1, 0, 2**31 - 1, -2**31], int(((odd > 0.08) & (odd < 0.12)).sum()))
    acc = np.clip(acc, -2**31, 2**31 - 1)
    return tuple(x.astype(np.int32) for x in (task, slo, acc, bidx))


@pytest.mark.parametrize("kind", ["stairs", "mixed", "noisy", "wide"])
@pytest.mark.parametrize("lengths", [(n, 5, n - 1, 0, n) for n in LENGTHS] + [(70_000,)], ids=lambda v: str(v[0]))
def test_ranked_slices(oracle_lib, kind, lengths):
    rng = np.random.default_rng(lengths[0] * 7 + len(kind))
    B = 1 if lengths[0] > 60_000 else 2
    tb = _ranked_table(kind, lengths, B, rng)
    n = 700 if lengths[0] > 60_000 else 4001
    qs = _ranked_queries(tb, n, rng)
    sel = make_selector(tb, engine=0)
    print(f"ranked {kind} {lengths}: truncated {sel.info()['index_truncated']} of {tb.num_tasks * B}", flush=True)
    queue = tb.queue_us.copy()
    for rnd in range(2):
        if rnd:   # a report on a third of the variants; the nodes are written anew
            rows = rng.choice(tb.V, tb.V // 3, replace=False).astype(np.int32)
            vals = rng.integers(0, 30_000, rows.size).astype(np.int32)
            sel.update_load(to_dev(rows), to_dev(vals))
            oracle_lib.update_load(queue, rows, vals)
        got = gpu_select(sel, *qs)
        want = oracle_lib.select(*table_args(tb, queue), *qs)
        _assert_equal_everywhere(got, want, f"{kind} {lengths} round {rnd}")
        assert (want >= 0).sum() > n // 10
    sel.destroy()


@pytest.mark.parametrize("kind", ["noisy", "mixed"])
def test_ranked_batches_and_short_rests(oracle_lib, kind):
    """Batch sizes around those at which a wavefront takes more queries (powers of two times two wavefronts per
    SIMD: 2048 on 256 compute units), and slices of which 256 or 512 entries, or a few more or fewer, are left behind
    the first 16."""
    rng = np.random.default_rng(17)
    tb = _ranked_table(kind, (272, 271, 273, 276, 528, 527, 529, 532, 100), 2, rng)
    qs = _ranked_queries(tb, 131_073, rng)
    want = oracle_lib.select(*table_args(tb), *qs)
    sel = make_selector(tb, engine=0)
    assert sel.info()["index_truncated"] > tb.num_tasks
    for n in (1, 2, 3, 2047, 2048, 2049, 4095, 4097, 8193, 16385, 32767, 65537, 131_072, 131_073):
        _assert_equal_everywhere(gpu_select(sel, *(x[:n] for x in qs)), want[:n], f"{kind} N={n}")
    sel.destroy()


@pytest.mark.parametrize("kind", ["stairs", "mixed", "noisy", "wide"])
def test_ranked_many_slices(oracle_lib, kind):
    """More than 512 slices in one pool (built one per wavefront), most of them truncated, a few of them long enough for
    sorted blocks and for levels above the first."""
    rng = np.random.default_rng(23)
    T = 300
    lengths = rng.integers(64, 150, T)
    lengths[[0, 5, 100, 101, 299]] = (4097, 529, 600, 1025, 2000)
    tb = _ranked_table(kind, tuple(int(n) for n in lengths), 2, rng)
    qs = _ranked_queries(tb, 60_001, rng)
    long = rng.random(60_001) < 0.4
    qs[0][long] = rng.choice(np.asarray([0, 5, 100, 101, 299], np.int32), int(long.sum()))
    sel = make_selector(tb, engine=0)
    queue = tb.queue_us.copy()
    for rnd in range(2):
        if rnd:
            rows, vals = rng.choice(tb.V, tb.V // 3, replace=False).astype(np.int32), rng.integers(0, 30_000, tb.V // 3).astype(np.int32)
            sel.update_load(to_dev(rows), to_dev(vals))
            oracle_lib.update_load(queue, rows, vals)
        want = oracle_lib.select(*table_args(tb, queue), *qs)
        for part in (slice(0, 2001), slice(None)):
            _assert_equal_everywhere(gpu_select(sel, *(x[part] for x in qs)), want[part], f"{kind} round {rnd}")
    sel.destroy()


@pytest.mark.parametrize("T,B", [(20, 4), (130, 4)])
def test_ranked_two_tiers(oracle_lib, T, B):
    """Truncated slices in both tiers, up to 600 entries of either state: the nodes of two tables written by one
    launch, one slice per workgroup and (more than 1024 slices) one per wavefront; masked entries in every sorted block."""
    rng = np.random.default_rng(T)
    lengths = [80] * T
    lengths[0], lengths[3], lengths[T - 1] = 1300, 1100, 2100
    tb = _ranked_table("noisy", tuple(lengths), B, rng)
    state, load = rng.integers(0, 3, tb.V).astype(np.int32), rng.integers(100, 60_000, tb.V).astype(np.int32)
    qs = _ranked_queries(tb, 20_003, rng)
    long = rng.random(20_003) < 0.5
    qs[0][long] = rng.choice(np.asarray([0, 3, T - 1], np.int32), int(long.sum()))
    sel = make_selector(tb, engine=0)
    sel.load_states(state, load)
    state = state.copy()
    for rnd in range(2):
        if rnd:
            rows, vals = rng.choice(tb.V, tb.V // 2, replace=False).astype(np.int32), rng.integers(0, 3, tb.V // 2).astype(np.int32)
            sel.update_state(to_dev(rows), to_dev(vals))
            oracle_lib.update_state(state, rows, vals)
        for g, w in zip(gpu_select_tiered(sel, *qs), oracle_lib.select_tiered(*table_args(tb), state, load, *qs)):
            _assert_equal_everywhere(g, w, f"tiers round {rnd}")
        for g, w in zip(gpu_case1(sel, *qs), oracle_lib.select_case1(*table_args(tb), state, load, *qs)):
            _assert_equal_everywhere(g, w, f"case I round {rnd}")
    sel.destroy()


@pytest.mark.parametrize("span", [0xFFFFFD, 0xFFFFFE, 0xFFFFFF, 0x1000000])
@pytest.mark.parametrize("low", [-2**31, -2**31 + 1, -5, 2**31 - 1 - 0x1000000])
def test_ranked_accuracies_around_24_bits(oracle_lib, low, span):
    """Sorted blocks are made from accuracies counted in 24 bits where they fit, and as they are where not."""
    rng = np.random.default_rng(span & 0xFF)
    tb = _ranked_table("noisy", (600, 900), 2, rng)
    acc = (low + np.floor((tb.acc_bp - 5000) / 9000 * span)).astype(np.int64)
    acc[np.flatnonzero(tb.task_id == 0)[[7, 300]]] = (low, low + span)
    acc[np.flatnonzero(tb.task_id == 1)[[800, 2]]] = (low, low + span)
    tb = _table(2, tb.batch_sizes, tb.task_id, acc, tb.lat_us, tb.cost, tb.queue_us)
    qs = _ranked_queries(tb, 20_001, rng)
    sel = make_selector(tb, engine=0)
    assert sel.info()["index_truncated"] == 4
    _assert_equal_everywhere(gpu_select(sel, *qs), oracle_lib.select(*table_args(tb), *qs), f"{low} + {span}")
    sel.destroy()
