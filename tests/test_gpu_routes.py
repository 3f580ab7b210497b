"""Calls beyond the old limits that a lane per query still answers, and those behind them: both sides of the lines
that the shape of the index draws, with every element against the CPU oracle."""
import numpy as np
import pytest

import workloads
from gpu_util import gpu_select, gpu_select_closest, make_selector, query_args, table_args
from test_gpu_direct import TABLES
from test_gpu_parity import _assert_equal_everywhere
from test_gpu_tiered import gpu_select_tiered

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", list(TABLES))
def test_selections_and_suggestions_of_every_size(oracle_lib, kind):
    """From the sizes that count every query as parked to those that the mirror or a tile at a time answers, on an index that fits
    the mirror, one that does in part, one in groups and one without a mirror."""
    tb = TABLES[kind]()
    rng = np.random.default_rng(17)
    q = workloads.make_queries(1, n=70_001, seed=5)
    qs = (rng.integers(0, tb.num_tasks, q.N).astype(np.int32), *query_args(q)[1:3], rng.integers(0, tb.B, q.N).astype(np.int32))
    want, closest = oracle_lib.select_closest(*table_args(tb), *qs)
    sel = make_selector(tb, engine=2)
    for n in (110_003, 349_999, 350_001, 600_001, 899_999, 900_001, 1_400_003):
        many = [np.tile(x, n // q.N + 1)[:n] for x in (*qs, want, closest)]
        _assert_equal_everywhere(gpu_select(sel, *many[:4]), many[4], f"{kind} N={n}")
        for got, w in zip(gpu_select_closest(sel, *many[:4]), many[4:]):
            _assert_equal_everywhere(got, w, f"{kind} closest N={n}")
    sel.destroy()


def test_two_tiers_of_every_size(oracle_lib):
    tb = workloads.make_table(0)
    st = workloads.make_states(0, tb.V)
    q = tuple(x[:10_000] for x in query_args(workloads.make_queries(0)))
    want = oracle_lib.select_tiered(*table_args(tb), st.state, st.load_us, *q)
    sel = make_selector(tb, engine=0)
    sel.load_states(st.state, st.load_us)
    for n in (260_001, 800_003, 1_549_999, 1_550_001, 1_800_003):
        many = [np.tile(x, n // 10_000 + 1)[:n] for x in (*q, *want)]
        for got, w in zip(gpu_select_tiered(sel, *many[:4]), many[4:]):
            _assert_equal_everywhere(got, w, f"two tiers N={n}")
    sel.destroy()
