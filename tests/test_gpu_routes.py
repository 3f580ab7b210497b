"""Which way a call goes: the sizes on both sides of the line between a lane per query and the mirror (or a tile at a time), for every
call and for tables that move the line, with every element against the CPU oracle."""
import numpy as np
import pytest

import workloads
from gpu_util import MEMORY, MIRROR, TILES, Repeated, make_selector, query_args, table_args
from test_gpu_direct import TABLES
from test_gpu_workers import cluster_args, load_cluster

pytestmark = pytest.mark.gpu

CALLS = ["select", "select_closest", "select_tiered", "select_tiered_closest", "select_workers", "select_workers_closest"]


def _handle(oracle_lib, call, tb, cfg, qs):
    """A handle that is ready for the call, and the oracle's results."""
    sel = make_selector(tb, engine=2)
    if call == "select":
        return sel, [oracle_lib.select(*table_args(tb), *qs)]
    if call == "select_closest":
        return sel, oracle_lib.select_closest(*table_args(tb), *qs)
    st = workloads.make_states(cfg, tb.V)
    sel.load_states(st.state, st.load_us)
    args = (*table_args(tb), st.state, st.load_us)
    if "workers" in call:
        cl = cluster_args(workloads.make_workers(cfg, st))
        load_cluster(sel, cl)
        args += cl
    return sel, {"select_tiered": oracle_lib.select_tiered, "select_tiered_closest": oracle_lib.select_case1,
                 "select_workers": oracle_lib.select_workers, "select_workers_closest": oracle_lib.get_variant}[call](*args, *qs)


@pytest.mark.parametrize("call", CALLS)
@pytest.mark.parametrize("cfg", [0, 1, 2])
def test_both_sides_of_the_line(oracle_lib, call, cfg):
    """An index that fits the mirror several times over, one that does so all but a tenth, and one that just does."""
    tb = workloads.make_table(cfg)
    qs = tuple(x[:30_011] for x in query_args(workloads.make_queries(cfg)))
    sel, want = _handle(oracle_lib, call, tb, cfg, qs)
    many = Repeated(sel, getattr(sel, call), qs, want)
    many.route(1)     # (the sizes of the tiers' own indexes are known to the host from the first call on)
    limit = many.last_from_memory(8_000_001)
    beyond = TILES if (call, cfg) == ("select", 1) else MIRROR
    assert 100_000 < limit < 6_000_000
    for n, route in ((limit, MEMORY), (limit + 1, beyond), (limit * 5 // 4, beyond)):
        many.check(n, route, f"{call} config {cfg}")
    sel.destroy()


@pytest.mark.parametrize("call", CALLS)
@pytest.mark.parametrize("kind", ["groups", "no_mirror"])
def test_tables_that_the_mirror_does_not_pay_for(oracle_lib, call, kind):
    """Most bodies outside the mirror, or none in it: straight from memory at every size, the plain selection a tile at a time."""
    tb = TABLES[kind]()
    rng = np.random.default_rng(17)
    q = workloads.make_queries(1, n=30_011, seed=5)
    qs = (rng.integers(0, tb.num_tasks, q.N).astype(np.int32), *query_args(q)[1:3], rng.integers(0, tb.B, q.N).astype(np.int32))
    sel, want = _handle(oracle_lib, call, tb, 3, qs)
    many = Repeated(sel, getattr(sel, call), qs, want)
    for n in (1_499_999, 1_500_000, 3_000_001):
        many.check(n, TILES if call == "select" and n >= 1_500_000 else MEMORY, f"{call} {kind}")
    sel.destroy()
