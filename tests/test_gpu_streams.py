"""Two handles with different tables working at the same time on two streams: every answer against the
CPU oracle.  A handle owns its table, index and scratch memory, so handles do not have to be ordered
with each other (only infaas_sel_select_noalloc shares memory between handles)."""
import ctypes
import threading

import numpy as np
import pytest

import workloads
from gpu_util import make_selector, query_args, table_args, to_dev

pytestmark = pytest.mark.gpu


def test_two_handles_on_two_streams(oracle_lib):
    import torch
    cfgs, n, rounds = (1, 4), 600_000, 3
    tabs = [workloads.make_table(c) for c in cfgs]
    sels = [make_selector(tb, engine=0) for tb in tabs]
    for sel in sels:
        sel.reserve(n)
    streams = [torch.cuda.Stream() for _ in cfgs]
    queues = [tb.queue_us.copy() for tb in tabs]
    batches = [[workloads.make_queries(c, n=n, chunk=r) for r in range(rounds)] for c in cfgs]
    reports = [[workloads.make_load_update(c, tb.V, r + 1) for r in range(rounds)] for c, tb in zip(cfgs, tabs)]
    dev_q = [[[to_dev(x) for x in query_args(q)] for q in qs] for qs in batches]
    dev_r = [[(to_dev(u.variant_idx), to_dev(u.queue_us)) for u in us] for us in reports]
    outs = [[torch.full((n,), -777, dtype=torch.int32, device="cuda") for _ in range(rounds)] for _ in cfgs]
    torch.cuda.synchronize()
    # report, select, report, select ... on each handle's own stream, the two streams interleaved
    for r in range(rounds):
        for k in range(2):
            with torch.cuda.stream(streams[k]):
                sels[k].update_load(*dev_r[k][r])
                sels[k].select(*dev_q[k][r], outs[k][r])
    torch.cuda.synchronize()
    for k, (c, tb) in enumerate(zip(cfgs, tabs)):
        for r in range(rounds):
            oracle_lib.update_load(queues[k], reports[k][r].variant_idx, reports[k][r].queue_us)
            print(f"two streams: config {c} round {r}", flush=True)
            want = oracle_lib.select(*table_args(tb, queues[k]), *query_args(batches[k][r]))
            got = outs[k][r].cpu().numpy()
            bad = np.flatnonzero(got != want)
            assert bad.size == 0, f"config {c} round {r}: {bad.size} differ, first at {bad[:5]}"
    for sel in sels:
        sel.destroy()


def _thread_local_data(library):
    """Address of the calling thread's thread-local data of a loaded library; 0 while the thread has read none of it."""
    class Info(ctypes.Structure):
        _fields_ = [("addr", ctypes.c_size_t), ("name", ctypes.c_char_p), ("phdr", ctypes.c_void_p), ("phnum", ctypes.c_uint16),
                    ("adds", ctypes.c_ulonglong), ("subs", ctypes.c_ulonglong), ("tls_module", ctypes.c_size_t), ("tls_data", ctypes.c_size_t)]
    found = []

    @ctypes.CFUNCTYPE(ctypes.c_int, ctypes.POINTER(Info), ctypes.c_size_t, ctypes.c_void_p)
    def look(info, size, data):
        if info.contents.name.endswith(library.encode()):
            found.append((info.contents.tls_module, info.contents.tls_data))
        return 0
    ctypes.CDLL(None).dl_iterate_phdr(look, None)
    assert len(found) == 1 and found[0][0] > 0
    return found[0][1]


@pytest.mark.parametrize("call", ["select", "update_load"])
def test_a_call_brings_its_threads_storage_up_to_date(call):
    """A thread that has called the library has read a thread-local variable of it (without which every other library's cost it more)."""
    import torch
    tb = workloads.make_table(0)
    sel = make_selector(tb, engine=0)
    dev = [to_dev(x[:1000]) for x in query_args(workloads.make_queries(0))]
    out = torch.empty_like(dev[0])
    rows = to_dev(np.arange(10))
    seen = []

    def work():
        seen.append(_thread_local_data("libinfaas_sel.so"))
        sel.select(*dev, out) if call == "select" else sel.update_load(rows, rows)
        seen.append(_thread_local_data("libinfaas_sel.so"))
    thread = threading.Thread(target=work)
    thread.start()
    thread.join()
    torch.cuda.synchronize()
    assert len(seen) == 2 and seen[0] == 0 and seen[1] != 0
    sel.destroy()
