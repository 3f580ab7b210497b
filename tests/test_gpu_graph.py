"""The calls that enqueue work allocate nothing and synchronise nothing once their scratch memory
exists, so a caller may capture them into a HIP graph.  Each graph is replayed several times with
new contents in its input buffers and eager work in between, and every replay is checked against
the CPU oracle."""
import numpy as np
import pytest

import workloads
from gpu_util import MEMORY, MIRROR, make_selector, table_args, to_dev

pytestmark = pytest.mark.gpu


def _capture(fn):
    """Warm up on a side stream, then capture fn() into a graph."""
    import torch
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        fn()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        fn()
    return g


def _fill(dst, src):
    import torch
    for d, x in zip(dst, src):
        d.copy_(torch.from_numpy(np.ascontiguousarray(x, dtype=np.int32)))


def test_graph_load_report_and_select(oracle_lib):
    import torch
    cfg, n = 1, 200_000
    tb = workloads.make_table(cfg)
    sel = make_selector(tb, engine=0)
    qs = [workloads.make_queries(cfg, n=n, chunk=c) for c in range(3)]
    ups = [workloads.make_load_update(cfg, tb.V, c + 1) for c in range(3)]
    dq = [torch.empty(n, dtype=torch.int32, device="cuda") for _ in range(4)]
    du = [torch.empty(ups[0].variant_idx.size, dtype=torch.int32, device="cuda") for _ in range(2)]
    out = torch.empty(n, dtype=torch.int32, device="cuda")
    clo = torch.empty_like(out)

    def step():
        sel.update_load(*du)
        sel.select_closest(*dq, out, clo)

    _fill(dq, (qs[0].task, qs[0].slo_us, qs[0].min_acc_bp, qs[0].batch_idx))
    _fill(du, (ups[0].variant_idx, ups[0].queue_us))
    graph = _capture(step)
    queue = tb.queue_us.copy()
    oracle_lib.update_load(queue, ups[0].variant_idx, ups[0].queue_us)       # applied by the warm-up and the capture run
    for rep in range(6):
        i = rep % 3
        q = qs[i]
        _fill(dq, (q.task, q.slo_us, q.min_acc_bp, q.batch_idx))
        _fill(du, (ups[i].variant_idx, ups[i].queue_us))
        out.fill_(-9); clo.fill_(-9)
        assert int((out + 1).sum().item()) == -8 * n                         # eager work between the replays
        graph.replay()
        torch.cuda.synchronize()
        oracle_lib.update_load(queue, ups[i].variant_idx, ups[i].queue_us)
        want = oracle_lib.select_closest(*table_args(tb, queue), q.task, q.slo_us, q.min_acc_bp, q.batch_idx)
        print(f"graph replay {rep}", flush=True)
        assert np.array_equal(out.cpu().numpy(), want[0]) and np.array_equal(clo.cpu().numpy(), want[1]), f"replay {rep}"
    sel.destroy()


def test_graph_reports_workers_and_scaling(oracle_lib):
    """State report, worker report, the selection with workers and a batch of scaling decisions, up
    and down, in one graph."""
    import torch
    cfg, n, r = 1, 150_000, 50_000
    tb = workloads.make_table(cfg)
    st = workloads.make_states(cfg, tb.V)
    wk = workloads.make_workers(cfg, st)
    sc = workloads.make_scaling(cfg, tb)
    sel = make_selector(tb, engine=0)
    sel.load_states(st.state, st.load_us)
    sel.load_workers(wk.worker_hw, wk.worker_util, wk.variant_hw, wk.inst_variant, wk.inst_worker, wk.inst_load)
    sel.load_scaling(sc.arch_id, sc.sat_qps, sc.hw_cost, sc.load_us, 50, 105)
    sel.reserve(n)                                                            # the lists of open queries
    qs = [workloads.make_queries(cfg, n=n, chunk=c) for c in range(2)]
    sus = [workloads.make_state_update(cfg, tb.V, c + 1) for c in range(2)]
    wus = [workloads.make_worker_update(cfg, wk.W, wk.I, c + 1) for c in range(2)]
    rqs = [workloads.make_scale_requests(cfg, tb, sc, r, chunk=c) for c in range(2)]
    dq = [torch.empty(n, dtype=torch.int32, device="cuda") for _ in range(4)]
    ds = [torch.empty(sus[0].variant_idx.size, dtype=torch.int32, device="cuda") for _ in range(2)]
    dw = [torch.empty(x.size, dtype=torch.int32, device="cuda") for x in
          (wus[0].worker_idx, wus[0].worker_util, wus[0].inst_idx, wus[0].inst_load)]
    dr = [torch.empty(r, dtype=torch.int32, device="cuda") for _ in range(5)]
    res = [torch.empty(n, dtype=torch.int32, device="cuda") for _ in range(3)]
    dec = [torch.empty(r, dtype=torch.int32, device="cuda") for _ in range(3)]
    dec_down = [torch.empty(r, dtype=torch.int32, device="cuda") for _ in range(3)]

    def step():
        sel.update_state(*ds)
        sel.update_workers(*dw)
        sel.select_workers(*dq, *res)
        sel.scale(*dr, *dec)
        sel.scale_down(*dr, *dec_down)

    def stage(i):
        q, su, wu, rq = qs[i], sus[i], wus[i], rqs[i]
        _fill(dq, (q.task, q.slo_us, q.min_acc_bp, q.batch_idx))
        _fill(ds, (su.variant_idx, su.state))
        _fill(dw, (wu.worker_idx, wu.worker_util, wu.inst_idx, wu.inst_load))
        _fill(dr, (rq.variant, rq.instances, rq.load_qps, rq.slo_us, rq.batch_idx))

    state, util, iload = st.state.copy(), wk.worker_util.copy(), wk.inst_load.copy()

    def apply(i):
        oracle_lib.update_state(state, sus[i].variant_idx, sus[i].state)
        oracle_lib.update_worker_util(util, wus[i].worker_idx, wus[i].worker_util)
        oracle_lib.update_instance_load(iload, wus[i].inst_idx, wus[i].inst_load)

    stage(0)
    graph = _capture(step)
    apply(0)
    for rep in range(5):
        i = rep % 2
        stage(i)
        for t in res + dec + dec_down:
            t.fill_(-9)
        assert int((res[0] + 1).sum().item()) == -8 * n
        graph.replay()
        torch.cuda.synchronize()
        apply(i)
        q, rq = qs[i], rqs[i]
        want = oracle_lib.select_workers(*table_args(tb), state, st.load_us, wk.variant_hw, wk.worker_hw, util,
                                         wk.inst_variant, wk.inst_worker, iload, q.task, q.slo_us, q.min_acc_bp,
                                         q.batch_idx)
        want_dec = oracle_lib.scale(sc.arch_id, sc.sat_qps, sc.hw_cost, sc.load_us, tb.lat_us, 50, 105, rq.variant,
                                    rq.instances, rq.load_qps, rq.slo_us, rq.batch_idx)
        want_down = oracle_lib.scale_down(sc.arch_id, sc.sat_qps, sc.hw_cost, sc.load_us, tb.lat_us, 50, 105, rq.variant,
                                          rq.instances, rq.load_qps, rq.slo_us, rq.batch_idx)
        print(f"graph replay {rep}", flush=True)
        for g, w in zip(res + dec + dec_down, want + want_dec + want_down):
            assert np.array_equal(g.cpu().numpy(), w), f"replay {rep}"
    sel.destroy()


class _Cluster:
    """A handle with workers (and instance states) beside a host copy of everything reports change, and one report of each
    kind at a time on both."""

    def __init__(self, oracle_lib, instances, n=5003, cfg=1):
        self.lib, self.cfg, self.n, self.turn = oracle_lib, cfg, n, 0
        times = 900                               # 4,502,700 queries go through the LDS mirrors, 5003 straight from memory
        self.tb = workloads.make_table(cfg)
        self.st = workloads.make_states(cfg, self.tb.V)
        self.wk = workloads.make_workers(cfg, self.st)
        self.state, self.queue = self.st.state.copy(), self.tb.queue_us.copy()
        self.util, self.iload = self.wk.worker_util.copy(), self.wk.inst_load.copy()
        self.ist = workloads.make_instance_states(cfg, self.wk.I) if instances else None
        self.sel = make_selector(self.tb, engine=0)
        self.sel.load_states(self.state, self.st.load_us)
        self.load_workers()
        q = workloads.make_queries(cfg, n=n)
        self.q = (q.task, q.slo_us, q.min_acc_bp, q.batch_idx)
        self.dq, self.out = [to_dev(np.tile(x, times)) for x in self.q], [to_dev(np.zeros(n * times)) for _ in range(3)]
        self.staged = {}

    def load_workers(self):
        w = self.wk
        self.sel.load_workers(w.worker_hw, self.util, w.variant_hw, w.inst_variant, w.inst_worker, self.iload)
        if self.ist is not None:
            self.sel.load_instance_states(self.ist)

    def stage(self, kind):
        """New contents for the device buffers of a report of this kind; what the device will hold once it has run."""
        self.turn += 1
        w, V, lib = self.wk, self.tb.V, self.lib
        if kind == "load":
            u = workloads.make_load_update(self.cfg, V, self.turn)
            host = (u.variant_idx, u.queue_us)
            lib.update_load(self.queue, *host)
        elif kind == "state":
            u = workloads.make_state_update(self.cfg, V, self.turn, fraction=0.3)
            host = (u.variant_idx, u.state)
            lib.update_state(self.state, *host)
        elif kind == "workers":
            u = workloads.make_worker_update(self.cfg, w.W, w.I, self.turn, fraction=0.5)
            host = (u.worker_idx, u.worker_util, u.inst_idx, u.inst_load)
            lib.update_worker_util(self.util, *host[:2])
            lib.update_instance_load(self.iload, *host[2:])
        else:
            host = workloads.make_instance_state_update(self.cfg, w.I, self.turn, fraction=0.3)
            lib.update_instance_state(self.ist, *host)
        if kind not in self.staged:
            self.staged[kind] = [to_dev(x) for x in host]
        _fill(self.staged[kind], host)

    def report(self, kind):
        call = {"load": self.sel.update_load, "state": self.sel.update_state, "workers": self.sel.update_workers,
                "instances": self.sel.update_instance_states}[kind]
        call(*self.staged[kind])

    def now(self, kind):
        self.stage(kind)
        self.report(kind)

    def select(self):
        self.sel.select_workers(*self.dq, *self.out)

    def check(self, label, size=None):
        import torch
        size = size or self.out[0].numel()
        torch.cuda.synchronize()
        print(f"workers {label}", flush=True)
        w = self.wk
        tables = (*table_args(self.tb, self.queue), *(() if self.ist is not None else (self.state,)), self.st.load_us,
                  w.variant_hw, w.worker_hw, self.util, w.inst_variant, w.inst_worker, self.iload)
        want = self.lib.select_workers(*tables, *self.q) if self.ist is None else self.lib.select_instances(*tables, self.ist, *self.q)
        for got, x, what in zip(self.out, want, ("variant", "tier", "worker")):
            got = got.cpu().numpy()[:size]
            assert np.array_equal(got, np.tile(x, size // self.n)), f"{label}: {what}"

    def select_and_check(self, label):
        for size in (self.n, self.out[0].numel()):
            for o in self.out:
                o.fill_(-9)
            self.sel.select_workers(*self.dq, *self.out, n=size)
            self.check(f"{label}, {size} queries", size)
            assert self.sel.info()["lookup_route"] == (MEMORY if size == self.n else MIRROR)


def _record(fn):
    import torch
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        fn()
    return g


@pytest.mark.parametrize("between", ["nothing", "state", "load", "reload"])
def test_a_recorded_refresh_has_not_happened(oracle_lib, between):
    """A selection with workers that is recorded behind a worker report, but not replayed yet, has brought nothing up to
    date: neither for an eager call nor for the build behind a state report, nor for the graph of another selection."""
    c = _Cluster(oracle_lib, instances=False)
    c.select_and_check("eager")
    for rnd in range(3):
        if between == "reload":
            c.load_workers()
        else:
            c.now("workers")
        graph = _record(lambda: (c.select(), c.select()))
        other = _record(c.select)
        if between in ("state", "load"):
            c.now(between)
        if rnd < 2:
            c.select_and_check(f"eager behind a recorded selection, round {rnd}")
        if between in ("nothing", "reload"):    # (behind a report a selection is recorded again)
            for g, what in ((other, "second"), (graph, "first"), (other, "second again")):
                for o in c.out:
                    o.fill_(-9)
                g.replay()
                c.check(f"the {what} graph, round {rnd}")
        c.select_and_check(f"eager behind the replays, round {rnd}")
    c.sel.destroy()


@pytest.mark.parametrize("kind,instances", [("load", False), ("state", False), ("workers", False), ("workers", True), ("instances", True)])
def test_graph_of_a_report_alone(oracle_lib, kind, instances):
    """A report recorded without a selection: an eager selection with workers answers by it behind every replay, whatever
    was reported and selected eagerly in between."""
    c = _Cluster(oracle_lib, instances)
    c.select_and_check("eager")
    c.now(kind)
    graph = _record(lambda: c.report(kind))
    for rnd in range(4):
        eager = kind if rnd % 2 == 0 else ("instances" if instances else "state")
        c.now(eager)
        if rnd >= 2:
            c.select_and_check(f"{kind}, eager {eager}, round {rnd}")
        c.stage(kind)
        graph.replay()
        c.select_and_check(f"{kind}, replay {rnd}")
    c.sel.destroy()


def test_graph_of_instance_state_reports(oracle_lib):
    """Worker and instance state report and the selection with workers in one graph, replayed between eager reports of both
    kinds and eager selections."""
    c = _Cluster(oracle_lib, instances=True)

    def step():
        c.report("workers")
        c.report("instances")
        c.select()

    c.stage("workers")
    c.stage("instances")
    graph = _capture(step)                      # (the warm-up and the recorded step carry the same report)
    for rnd in range(6):
        if rnd % 3 == 1:
            c.now("instances")
            c.select_and_check(f"eager, round {rnd}")
        elif rnd % 3 == 2:
            c.now("instances")
            c.now("workers")
        c.stage("workers")
        c.stage("instances")
        for o in c.out:
            o.fill_(-9)
        graph.replay()
        c.check(f"replay {rnd}")
        if rnd % 2:
            c.select_and_check(f"eager behind replay {rnd}")
    c.sel.destroy()
