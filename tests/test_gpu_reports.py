"""State reports applied to both tiers' tables in one launch (64 / B entries of a report per wavefront) and
both indexes built in one: batch-size counts that divide 64 and that do not, slices around the sizes of the
build's chunks (256, 512, 1024, 2048 entries), reports that change a state, repeat it, or must be
skipped; every element of variant, tier and worker against the CPU oracle."""
import numpy as np
import pytest

from gpu_util import gpu_select, make_selector, table_args, to_dev
from test_gpu_instances import _check as check_instances
from test_gpu_parity import _assert_equal_everywhere, _random_queries, _random_table, _table
from test_gpu_workers import _check as check_workers, _random_cluster, load_cluster

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,sizes", [(1, (255, 256, 3)), (3, (257, 0, 40)), (5, (511, 512)), (7, (513, 1, 90)), (8, (64, 65, 1)),
                                     (33, (20, 31)), (64, (5, 33)), (2, (1024, 1025)), (2, (2048, 2049))],
                         ids=lambda v: str(v).replace(" ", ""))
def test_state_reports(oracle_lib, B, sizes):
    rng = np.random.default_rng(B * 1000 + sum(sizes))
    T = len(sizes)
    tb = _random_table(rng, T, np.asarray(sizes), min(B, 8))
    if B > 8:   # more batch sizes than the generator has: its columns over again, a little slower every time
        again = np.arange(B)
        tb = _table(T, list(range(1, B + 1)), tb.task_id, tb.acc_bp, tb.lat_us[:, again % 8] + again // 8, tb.cost[:, again % 8], tb.queue_us)
    state, load = rng.integers(0, 4, tb.V).astype(np.int32), rng.integers(0, 40_000, tb.V).astype(np.int32)
    cl = _random_cluster(rng, tb.V, state, 1000)
    qs = _random_queries(rng, T, B, 6000)
    sel = make_selector(tb, engine=0)
    sel.load_states(state, load)
    load_cluster(sel, cl)
    state, queue = state.copy(), tb.queue_us.copy()
    for rnd in range(3):
        n = int(rng.integers(1, tb.V + 1))
        rows, vals = rng.choice(tb.V, n, replace=False).astype(np.int32), rng.integers(0, 4, n).astype(np.int32)
        keep = rng.random(n) < 0.3
        vals[keep] = state[rows[keep]]                      # reported, but not changed
        if n > 3:
            rows[:2], vals[2] = (-1, tb.V), 4               # skipped
        sel.update_state(to_dev(rows), to_dev(vals))
        oracle_lib.update_state(state, rows, vals)
        up, q = rng.choice(tb.V, tb.V // 2 + 1, replace=False).astype(np.int32), rng.integers(0, 50_000, tb.V // 2 + 1).astype(np.int32)
        sel.update_load(to_dev(up), to_dev(q))
        oracle_lib.update_load(queue, up, q)
        check_workers(oracle_lib, sel, tb, state, load, cl, qs, f"B={B} {sizes} states {rnd}", queue)
    ist = rng.choice([1, 2, 3], max(len(cl[3]), 1))[:len(cl[3])].astype(np.int32)
    sel.load_instance_states(ist)
    for rnd in range(2):
        check_instances(oracle_lib, sel, tb, load, cl, ist, qs, f"B={B} {sizes} instances {rnd}", queue)
        if not len(ist):
            break
        idx, val = rng.choice(len(ist), len(ist) // 3 + 1, replace=False).astype(np.int32), rng.integers(0, 4, len(ist) // 3 + 1).astype(np.int32)
        sel.update_instance_states(to_dev(idx), to_dev(val))
        ok = val >= 1
        ist[idx[ok]] = val[ok]
    sel.destroy()


def test_two_build_kernels_on_one_handle(oracle_lib):
    """1024 slices in groups with states: a load report builds one table (a slice per workgroup, which reads
    what every slice publishes under the number of the build), a state report builds two (a slice per
    wavefront).  A build of the first kind with nothing but the second kind between it and the one 4095
    builds ago, whose number it carries: staircases of one or no step then, full ones now."""
    rng = np.random.default_rng(8)
    T, n, B = 128, 2000, 8
    tb = _random_table(rng, T, np.full(T, n), B)
    state = np.zeros(tb.V, np.int32)
    state[np.unique(tb.task_id, return_index=True)[1]] = 1        # one Active variant per task
    load = rng.integers(0, 40_000, tb.V).astype(np.int32)
    sel = make_selector(tb, engine=0)
    assert sel.info()["index_groups"] > 1
    sel.load_states(state, load)
    rows, vals = np.arange(0, tb.V, 7, dtype=np.int32), rng.integers(0, 50_000, (tb.V + 6) // 7).astype(np.int32)
    queue = tb.queue_us.copy()
    oracle_lib.update_load(queue, rows, vals)
    qs = _random_queries(rng, T, B, 200_000)
    dev = [to_dev(x) for x in (rows, vals)]
    one, same = to_dev(np.zeros(1, np.int32)), to_dev(state[:1])
    everything, active = to_dev(np.arange(tb.V, dtype=np.int32)), to_dev(np.ones(tb.V, np.int32))
    sel.update_load(*dev)
    for _ in range(4093):
        sel.update_state(one, same)
    sel.update_state(everything, active)
    sel.update_load(*dev)
    got = gpu_select(sel, *qs)
    _assert_equal_everywhere(got, oracle_lib.select(*table_args(tb, queue), *qs), "after 4095 builds")
    sel.destroy()


@pytest.mark.parametrize("T,B", [(300, 2), (170, 6), (513, 1)])
def test_build_with_slices_around_the_largest_chunk(oracle_lib, T, B):
    """More than 512 slices, up to 1024 of them, in one pool: a slice per wavefront, entries 2048 at a time."""
    rng = np.random.default_rng(T)
    sizes = rng.integers(0, 30, T)
    sizes[[0, 3, 7, 50, 51, 100, T - 1]] = (2048, 2047, 2049, 1025, 1024, 4097, 5000)
    tb = _random_table(rng, T, sizes, B)
    qs = _random_queries(rng, T, B, 250_000)
    half = rng.random(250_000) < 0.5
    qs[0][half] = rng.choice(np.asarray([0, 3, 7, 50, 51, 100, T - 1], np.int32), int(half.sum()))
    sel = make_selector(tb, engine=0)
    assert sel.info()["index_groups"] == 1
    queue = tb.queue_us.copy()
    for rnd in range(3):
        if rnd:
            rows, vals = rng.choice(tb.V, tb.V // 3, replace=False).astype(np.int32), rng.integers(0, 50_000, tb.V // 3).astype(np.int32)
            sel.update_load(to_dev(rows), to_dev(vals))
            oracle_lib.update_load(queue, rows, vals)
        _assert_equal_everywhere(gpu_select(sel, *qs), oracle_lib.select(*table_args(tb, queue), *qs), f"T={T} B={B} round {rnd}")
    sel.destroy()
