"""Helpers of the GPU parity tests: move inputs to the device, call the library, bring results back."""
import numpy as np


def to_dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).cuda()


class DeviceQueries:
    def __init__(self, task, slo, min_acc, bidx):
        import torch
        self.task, self.slo, self.min_acc, self.bidx = (to_dev(x) for x in (task, slo, min_acc, bidx))
        self.out = torch.full((max(self.task.numel(), 1),), -12345, dtype=torch.int32, device="cuda")
        self.n = int(self.task.numel())


def gpu_select(sel, task, slo, min_acc, bidx):
    """Run infaas_sel_select on host arrays; returns the host result."""
    import torch
    dq = DeviceQueries(task, slo, min_acc, bidx)
    sel.select(dq.task, dq.slo, dq.min_acc, dq.bidx, dq.out, n=dq.n)
    torch.cuda.synchronize()
    return dq.out[:dq.n].cpu().numpy()


def make_selector(table, engine=0, lds_segment_limit=0):
    import paper_1905_13348_amd as lib
    sel = lib.Selector(table.num_tasks, table.batch_sizes, device=0, engine=engine,
                       lds_segment_limit=lds_segment_limit)
    sel.load_variants(table.task_id, table.acc_bp, table.lat_us, table.cost, table.queue_us)
    return sel


# ways of a lookup (INFAAS_SEL_ROUTE_*)
MEMORY, MIRROR, TILES = 1, 2, 3


class Repeated:
    """Queries over and over on the device, and a call of a handle on as many of them as asked for.  `want`: the oracle's
    results for the queries, one array per result array of the call."""

    def __init__(self, sel, call, queries, want):
        self.sel, self.call = sel, call
        self.queries, self.want = [to_dev(x) for x in queries], [to_dev(x) for x in want]

    def _many(self, x, n):
        return x.repeat(n // x.numel() + 1)[:n]

    def route(self, n, shift=0):
        """The call on n queries, from arrays that start `shift` elements into their allocations; which way it went."""
        import torch
        args = [torch.cat([x.new_zeros(shift), self._many(x, n)])[shift:] for x in self.queries]
        self.got = [torch.full((n + shift,), -7, dtype=torch.int32, device="cuda")[shift:] for _ in self.want]
        self.call(*args, *self.got, n=n)
        torch.cuda.synchronize()
        return self.sel.info()["lookup_route"]

    def check(self, n, route, label, shift=0):
        """... which has to be `route` (None: not a lane per query), with the oracle's answers everywhere."""
        import torch
        label = f"{label} N={n} shift={shift}"
        print(label, flush=True)
        taken = self.route(n, shift)
        assert taken != MEMORY if route is None else taken == route, f"{label}: route {taken}"
        for k, (got, want) in enumerate(zip(self.got, self.want)):
            bad = torch.nonzero(got != self._many(want, n)).flatten()
            assert bad.numel() == 0, f"{label}: result {k}: {bad.numel()} differ, first at {bad[:5].tolist()}"

    def last_from_memory(self, most):
        """The most queries that go a lane per query; the next goes another way.  `most` queries go another way, one does not."""
        lo, hi = 1, most
        assert self.route(lo) == MEMORY and self.route(hi) != MEMORY
        while hi - lo > 1:
            mid = (lo + hi) // 2
            lo, hi = (mid, hi) if self.route(mid) == MEMORY else (lo, mid)
        return lo

    def least_beyond(self, least, most, route=None):
        """A size from `least` on that goes `route` (None: not a lane per query)."""
        n = least
        while True:
            taken = self.route(n)
            if (taken != MEMORY) if route is None else taken == route:
                return n
            n = n * 3 // 2 + 1
            assert n <= most, f"{n} queries: still route {taken}"


def table_args(tb, queue=None):
    return (tb.task_id, tb.acc_bp, tb.lat_us, tb.cost, tb.queue_us if queue is None else queue)


def query_args(q):
    return (q.task, q.slo_us, q.min_acc_bp, q.batch_idx)


def gpu_select_closest(sel, task, slo, min_acc, bidx):
    """Run infaas_sel_select_closest on host arrays; returns (selection, suggestion) on the host."""
    import torch
    dq = DeviceQueries(task, slo, min_acc, bidx)
    closest = torch.full_like(dq.out, -54321)
    sel.select_closest(dq.task, dq.slo, dq.min_acc, dq.bidx, dq.out, closest, n=dq.n)
    torch.cuda.synchronize()
    return dq.out[:dq.n].cpu().numpy(), closest[:dq.n].cpu().numpy()
