// Worker selection (Section 4.1, Case I: the policy returns the variant and the worker that serves
// the query; Section 6.4 counts the choice of the worker as the second decision on the critical
// path).  An Active variant is served by the least-loaded worker that runs an instance of it, an
// Inactive one by the least-utilised worker that has its target hardware.
//
// The worker depends on the variant and its tier only, not on the query.  So these kernels keep a
// worker per variant up to date (k_worker_tables, from the reports applied by k_worker_report) and
// copy it next to every step of the staircase indexes (k_step_workers); the lookup kernel then
// fetches the worker of an answer with the same gather that fetches its row.  All of it is bound by
// launches and latency (a few hundred KB), hence two launches, as many as there are dependencies, and behind an instance state
// report one: k_update_state, which goes through the instances anyway, does what k_worker_tables does.
#include "internal.h"
#include "lookup_common.h"

#include <algorithm>

namespace infaas {

namespace {

constexpr int kThreads = 256;

// util[worker_idx[i]] = util_new[i] (i < n) and load of instance inst_idx[j] = load_new[j] (j < m);
// entries outside the tables or with a negative value are skipped; the indices must be distinct.
__global__ __launch_bounds__(kThreads) void k_worker_report(WorkerView wv, int32_t n, const int32_t *__restrict__ worker_idx,
                                                            const int32_t *__restrict__ util_new, int32_t m,
                                                            const int32_t *__restrict__ inst_idx,
                                                            const int32_t *__restrict__ load_new)
{
    const int32_t i = (int32_t)(blockIdx.x * kThreads + threadIdx.x);
    if (i < n) {
        const int32_t w = worker_idx[i], u = util_new[i];
        if ((uint32_t)w < (uint32_t)wv.W && u >= 0) wv.util[w] = u;
    } else if (i - n < m) {
        const int32_t j = inst_idx[i - n], l = load_new[i - n];
        if ((uint32_t)j < (uint32_t)wv.I && l >= 0) wv.inst_load[wv.inst_pos[j]] = l;
    }
}

// State of instance inst_idx[i] = state[i]; a loaded instance is Active (1), Overloaded (2) or Interfered (3).
__global__ __launch_bounds__(kThreads) void k_instance_state_report(WorkerView wv, int32_t n, const int32_t *__restrict__ inst_idx,
                                                                   const int32_t *__restrict__ state)
{
    const int32_t i = (int32_t)(blockIdx.x * kThreads + threadIdx.x);
    if (i >= n) return;
    const int32_t j = inst_idx[i], c = state[i];
    if ((uint32_t)j < (uint32_t)wv.I && c >= 1 && c <= 3) wv.inst_state[wv.inst_pos[j]] = c;
}

// The first H workgroups, one per hardware class: the worker with the smallest (utilisation, number).
// The others, one lane per variant: the worker of its instance with the smallest (load, worker) -- of its
// Active instances, when the instances carry states.
__global__ __launch_bounds__(kThreads) void k_worker_tables(WorkerView wv)
{
    if ((int32_t)blockIdx.x < wv.H) {
        best_of_class<kThreads>(wv, (int32_t)blockIdx.x);
        return;
    }
    uint64_t best = ~0ull;
    const int32_t v = (int32_t)((blockIdx.x - (uint32_t)wv.H) * kThreads + threadIdx.x);
    if (v >= wv.V) return;
    for (int32_t i = wv.inst_off[v]; i < wv.inst_off[v + 1]; ++i) {
        if (wv.inst_state && wv.inst_state[i] != 1) continue;
        best = lower(best, instance_key(wv, i));
    }
    wv.row_worker[v] = best != ~0ull ? (int32_t)(uint32_t)best : -1;
}

// Workgroups (x, 0) serve the Active tier's index, (x, 1) the Inactive tier's (step_worker null: left alone):
// the worker of every step in use, and of the hot steps once more in 16 bits, as the lookup kernel keeps them
// in LDS.  Entries of step_row that a slice reserved but could not fill hold no row: anything outside 0..V-1
// gets no worker.  Places past a slice's last step are never read by the lookup.  rows: the second half of
// row_worker as well, the best worker of every variant's hardware class.
__global__ __launch_bounds__(kThreads) void k_step_workers(WorkerView wv, IndexView ia, IndexView ib, int32_t num_slices, int rows)
{
    const bool second = blockIdx.y != 0;
    const uint32_t *ctrl = second ? ib.ctrl : ia.ctrl;
    const int32_t *step_row = second ? ib.step_row : ia.step_row;
    int32_t *step_worker = second ? ib.step_worker : ia.step_worker;
    uint16_t *hot_worker = second ? ib.hot_worker : ia.hot_worker;
    const uint4 *hdr = second ? ib.hdr : ia.hdr;
    const uint32_t cap = second ? ib.step_cap : ia.step_cap, hot_rows = second ? ib.hot_rows : ia.hot_rows;
    const uint32_t first = blockIdx.x * kThreads + threadIdx.x, stride = gridDim.x * kThreads;
    auto class_worker = [&](int32_t row) {
        const int32_t c = wv.var_cls[row];
        return c >= 0 ? wv.best_cls[c] : -1;
    };
    auto worker = [&](uint32_t at) {
        const int32_t row = step_row[at];
        return (uint32_t)row >= (uint32_t)wv.V ? -1 : second ? class_worker(row) : wv.row_worker[row];
    };
    if (second && rows)
        for (uint32_t v = first; v < (uint32_t)wv.V; v += stride) wv.row_worker[wv.V + v] = class_worker((int32_t)v);
    if (!step_worker) return;
    const uint32_t used = ctrl[kCtlSteps];   // entries of step_row in use (entry 0 included)
    for (uint32_t j = first; j < used && j < cap; j += stride) step_worker[j] = worker(j);
    if (!hot_worker) return;
    for (uint32_t i = first; i < (uint32_t)num_slices * hot_rows; i += stride) {
        const uint32_t s = i / hot_rows, step = i - s * hot_rows;
        const uint4 h = hdr[s];
        const uint32_t at = h.z + step;   // the slice's first entry in step_row / step_worker, plus the step
        const int32_t w = ((h.y & kHdrPark) || at >= cap) ? -1 : worker(at);
        hot_worker[i] = (uint32_t)w < 0xFFFFu ? (uint16_t)w : (uint16_t)0xFFFFu;
    }
}

}  // namespace

hipError_t launch_worker_report(const WorkerView &wv, int32_t n, const int32_t *worker_idx, const int32_t *util,
                                int32_t m, const int32_t *inst_idx, const int32_t *load, hipStream_t st,
                                const LaunchEvents *ev)
{
    const int64_t total = (int64_t)n + m;
    if (total <= 0) return hipSuccess;
    return launch_kernel(ev, k_worker_report, dim3((unsigned)((total + kThreads - 1) / kThreads)), dim3(kThreads), 0, st,
                         wv, n, worker_idx, util, m, inst_idx, load);
}

hipError_t launch_instance_state_report(const WorkerView &wv, int32_t n, const int32_t *inst_idx, const int32_t *state,
                                        hipStream_t st, const LaunchEvents *ev)
{
    if (n <= 0 || !wv.inst_state) return hipSuccess;
    return launch_kernel(ev, k_instance_state_report, dim3((unsigned)((n + kThreads - 1) / kThreads)), dim3(kThreads), 0, st,
                         wv, n, inst_idx, state);
}

hipError_t launch_worker_tables(const WorkerView &wv, hipStream_t st, const LaunchEvents *ev)
{
    const int64_t blocks = (int64_t)wv.H + ((int64_t)wv.V + kThreads - 1) / kThreads;
    if (blocks <= 0) return hipSuccess;
    return launch_kernel(ev, k_worker_tables, dim3((unsigned)blocks), dim3(kThreads), 0, st, wv);
}

hipError_t launch_step_workers(const WorkerView &wv, const IndexView *ia, const IndexView *ib, int32_t num_slices, bool rows,
                               hipStream_t st, const LaunchEvents *ev)
{
    // the number of steps in use is known on the device only; a slice has at most kIndexCap
    const int64_t work = std::max<int64_t>((int64_t)num_slices * kIndexCap, wv.V);
    const int64_t blocks = std::min<int64_t>((work + kThreads - 1) / kThreads, 1024);
    return launch_kernel(ev, k_step_workers, dim3((unsigned)std::max<int64_t>(blocks, 1), 2), dim3(kThreads), 0, st, wv,
                         ia ? *ia : IndexView{}, ib ? *ib : IndexView{}, num_slices, rows ? 1 : 0);
}

}  // namespace infaas
