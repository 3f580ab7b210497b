"""Batches small enough to be answered straight from global memory, one lane per query, on both sides of
the size where the LDS mirror takes over: an index that fits the mirror, one that does so in part, one
laid out in groups and one whose headers leave no room for a mirror; arrays that start 4 bytes into
their allocations.  Every answer against the CPU oracle."""
import numpy as np
import pytest

import workloads
from gpu_util import make_selector, query_args, table_args
from test_gpu_parity import _assert_equal_everywhere, _random_table

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
