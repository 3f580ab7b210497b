"""The lines of the index (16 steps each, in four planes): staircases that end at and around the ends of the
planes, and tables whose caller rows do not fit beside the accuracy keys.  Every answer against the CPU oracle."""
import numpy as np
import pytest

from gpu_util import MEMORY, TILES, Repeated, gpu_select_closest, make_selector, table_args
from test_gpu_parity import _assert_equal_everywhere, _staircase_queries, _staircase_table, _table
from test_gpu_workers import _random_cluster, load_cluster

pytestmark = pytest.mark.gpu


def _rows_beyond_the_entries(tb):
    """The same table behind one more task whose two variants spread the accuracies over 16 bits: 16 bits are left
    for rows, and there are more rows than that."""
    task = np.concatenate([tb.task_id, np.full(2, tb.num_tasks, np.int32)])
    return _table(tb.num_tasks + 1, tb.batch_sizes, task, np.concatenate([tb.acc_bp, [tb.acc_bp.min(), tb.acc_bp.min() + 60_000]]),
                  np.concatenate([tb.lat_us, np.full((2, tb.B), 1000)]), np.concatenate([tb.cost, np.full((2, tb.B), 5)]),
                  np.concatenate([tb.queue_us, [0, 0]]))


@pytest.mark.parametrize("rows", ["in_the_entries", "beyond"])
@pytest.mark.parametrize("steps", [15, 16, 17, 30, 31, 32, 46, 47, 48, 61, 62, 63])
def test_staircases_around_the_ends_of_the_planes(oracle_lib, steps, rows):
    """As many steps in every slice as fill a plane, one less and one more: a large batch (a tile per workgroup at a time),
    one of the least size that goes there, one less and a small one (one query per lane)."""
    rng = np.random.default_rng(steps)
    tb = _staircase_table(-(-70_000 // steps), steps, B=1)
    if rows == "beyond":
        tb = _rows_beyond_the_entries(tb)
    sel = make_selector(tb, engine=2)
    assert sel.info()["index_groups"] > 1 and sel.info()["index_max_steps"] == min(steps, 62)
    qs = _staircase_queries(rng, tb, 300_007, steps)
    want = oracle_lib.select(*table_args(tb), *qs)
    many = Repeated(sel, sel.select, qs, [want])
    for n, route in ((2_100_049, TILES), (1_500_000, TILES), (1_499_999, MEMORY), (60_001, MEMORY)):
        many.check(n, route, f"{steps} steps, rows {rows}")
    assert (want >= 0).any() and (want < 0).any()
    sel.destroy()


@pytest.mark.parametrize("rows", ["in_the_entries", "beyond"])
@pytest.mark.parametrize("steps", [15, 16, 17, 31, 32, 47, 48, 62, 63])
def test_suggestions_around_the_ends_of_the_planes(oracle_lib, steps, rows):
    """The closest variant from the lines: staircases of these lengths, bounds that leave every requirement, one or both
    missed, negative and largest bounds among them, and ties in accuracy and latency (an odd task has pairs of both).  Then every
    call in two tiers, whose indexes the build for two tables writes."""
    rng = np.random.default_rng(100 + steps)
    T = 6 if rows == "in_the_entries" else -(-70_000 // steps)
    tb = _staircase_table(T, steps, B=2)
    odd = tb.task_id % 2 == 1
    tb.acc_bp[odd] = tb.acc_bp[odd] // 20 * 20
    tb.lat_us[odd] = tb.lat_us[odd] // 2000 * 2000
    if rows == "beyond":
        tb = _rows_beyond_the_entries(tb)
    sel = make_selector(tb, engine=2)
    n = 20_011
    task, bidx = rng.integers(0, T, n), rng.integers(0, 2, n)
    acc = rng.choice([-2**31, 0, 900, 1000, 1300, 2000, 70_000, 2**31 - 1], n) + rng.integers(0, 2 * steps, n) * (rng.random(n) < 0.5)
    slo = rng.choice([-2**31, -1, 0, 1, 20_000, 60_000, 90_000, 2**31 - 1], n)
    slo = np.where((slo > 1) & (slo < 2**31 - 1), slo + rng.integers(-20_000, 20_000, n), slo)
    qs = tuple(np.asarray(np.clip(x, -2**31, 2**31 - 1), np.int32) for x in (task, slo, acc, bidx))
    Repeated(sel, sel.select_closest, qs, oracle_lib.select_closest(*table_args(tb), *qs)).check(n, MEMORY, f"{steps} steps")
    state = (tb.task_id // 2 % 2).astype(np.int32)               # whole staircases in either tier
    state[rng.random(tb.V) < 0.02] = 2
    load = rng.integers(0, 20_000, tb.V).astype(np.int32)
    cl = _random_cluster(rng, tb.V, state, 1000)
    sel.load_states(state, load)
    load_cluster(sel, cl)
    args = (*table_args(tb), state, load)
    for call, want in ((sel.select_tiered, oracle_lib.select_tiered(*args, *qs)), (sel.select_tiered_closest, oracle_lib.select_case1(*args, *qs)),
                       (sel.select_workers, oracle_lib.select_workers(*args, *cl, *qs)),
                       (sel.select_workers_closest, oracle_lib.get_variant(*args, *cl, *qs))):
        Repeated(sel, call, qs, want).check(n, MEMORY, f"{steps} steps {call.__name__}")
        assert (want[1] == 1).any()
    sel.destroy()


def test_latencies_that_read_like_the_end_of_a_line(oracle_lib):
    """Latency plus queue just below 2^32 at every step, the last of the first line among them."""
    n = 20
    i = np.arange(n)
    tb = _table(1, [1], np.zeros(n, np.int32), 1000 + 10 * i, np.full((n, 1), 2**31 - 1), (10 + i)[:, None], 2**31 - 1 - i)
    sel = make_selector(tb, engine=2)
    acc = np.asarray([0, 1000, 1095, 1150, 1155, 1190, 1200], np.int32)
    qs = (np.zeros(7, np.int32), np.full(7, 2**31 - 1, np.int32), acc, np.zeros(7, np.int32))
    for got, want in zip(gpu_select_closest(sel, *qs), oracle_lib.select_closest(*table_args(tb), *qs)):
        _assert_equal_everywhere(got, want, "latencies below 2^32")
    sel.destroy()
