// Host runtime of libinfaas_sel: handle, variant-store build, scratch, launch sequencing.
// The operation and its C ABI are specified in include/infaas_sel.h.
#include "infaas_sel.h"
#include "internal.h"

#include <algorithm>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <new>
#include <numeric>
#include <vector>

using namespace infaas;

namespace {

thread_local char g_last_error[320] = "";

// Records which HIP call failed and why; returns true when the call succeeded.
bool hip_ok(hipError_t e, const char *what)
{
    if (e == hipSuccess) return true;
    snprintf(g_last_error, sizeof(g_last_error), "%s: %s (%d)", what, hipGetErrorString(e), (int)e);
    (void)hipGetLastError();
    return false;
}
#define HIP_OK(call) hip_ok((call), #call)

struct DeviceGuard {
    int prev = -1;
    bool ok = true;
    explicit DeviceGuard(int dev)
    {
        // Every call that enqueues comes through here, and reads a thread-local variable: while a thread has not done that since
        // this library was loaded behind others, glibc goes its slow way (10 ns) each time that the thread reads one of theirs, and
        // PyTorch does for every attribute of a tensor.  10,000 queries called from Python 6.2 us, so 5.5.
        (void)*(const volatile char *)g_last_error;
        if (!HIP_OK(hipGetDevice(&prev))) { ok = false; return; }
        if (prev != dev && !HIP_OK(hipSetDevice(dev))) ok = false;
        target = dev;
    }
    ~DeviceGuard()
    {
        if (prev >= 0 && prev != target) (void)hipSetDevice(prev);
    }
    int target = -1;
};

struct TimedLaunch {
    int kid;
    hipEvent_t a, b;
};

// ---- scratch memory for infaas_sel_select_noalloc
// The lookup kernel keeps one queue of parked queries per wavefront; every other entry point takes
// them from a hipMalloc'ed block of the handle.  For callers that may not allocate, the same queues
// live in this array, which the code object brings with it: 256 workgroups x 16 wavefronts x 320
// records x 16 bytes.  Every device the library runs on holds its own copy until the process ends.
// Host code never passes the array's name to a kernel (on the host the name is only a stand-in for
// the symbol): static_scratch() looks the device address up once per device and hands that out.
constexpr int kStaticMaxCus = 256;
constexpr size_t kStaticScratchBytes = (size_t)kStaticMaxCus * 16 * 320 * 16;   // 20 MiB
static __device__ __align__(256) __attribute__((used)) unsigned char scratch[kStaticScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void *g_scratch_ptr[kMaxDevices] = {nullptr};

// Device address of `scratch` on device `dev`, which must be the current device.  Null on failure
// (the reason is then in infaas_sel_last_error()).
void *static_scratch(int dev)
{
    if (dev < 0 || dev >= kMaxDevices) return nullptr;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void *ptr = nullptr;
        if (!hip_ok(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)), "hipGetSymbolAddress(scratch)")) return nullptr;
        g_scratch_ptr[dev] = ptr;
    }
    return g_scratch_ptr[dev];
}

template <typename T>
hipError_t dev_alloc(T **p, size_t count)
{
    *p = nullptr;
    return hipMalloc((void **)p, std::max<size_t>(count, 1) * sizeof(T));
}

}  // namespace

struct infaas_sel {
    int32_t T = 0, B = 0, device = 0;
    uint32_t flags = 0;
    int32_t lds_limit = 4096;
    int num_cus = 256;
    std::vector<int32_t> batch_sizes;

    bool loaded = false;
    // variant store (device)
    int32_t V = 0, Vp = 0;
    int32_t *d_acc = nullptr, *d_queue = nullptr, *d_orig = nullptr, *d_lat = nullptr;
    uint32_t *d_rank = nullptr, *d_perm = nullptr;
    int32_t *d_seg_off = nullptr, *d_seg_len = nullptr, *d_slot_of = nullptr;
    int32_t *d_acc_r = nullptr, *d_orig_r = nullptr;
    int2 *d_row_entry = nullptr;
    uint32_t *d_tot_r = nullptr;
    int64_t table_bytes = 0;
    int32_t max_segment = 0, max_lds_segment = 0, wide_segments = 0;
    TableView tv{};
    // state-aware selection: this table then serves the Active variants, `inactive` (a handle of
    // its own, built from the same rows) the Inactive ones
    std::vector<int32_t> h_task, h_acc, h_lat;   // host copies of the static columns, for building `inactive`
    int32_t *d_state = nullptr;                  // [V] state per row (see TableView::state)
    infaas_sel *inactive = nullptr;
    int32_t *d_open = nullptr;                   // lists of the queries the Active tier leaves open (grows)
    int32_t *d_open_count = nullptr;             // [workgroups of the lookup kernel]
    int64_t open_queries = 0, open_bytes = 0;    // pass size d_open is good for; its size
    int64_t open_words = 0;                      // 32-bit words of the lists proper; the side lists, if any, follow them
    bool open_side = false;
    // scaling decisions
    ScaleView sv{};
    std::vector<void *> scale_mem;               // the device arrays sv points into
    bool scaling_loaded = false;
    // worker selection (on the handle the caller holds; the step_worker arrays hang off both indexes)
    WorkerView wv{};
    std::vector<void *> worker_mem;              // the device arrays wv points into
    bool workers_loaded = false, workers_dirty = false;   // (dirty: older than the latest report)
    bool rows_stale = false;                              // the Inactive half of wv.row_worker is older than the workers
    bool instance_states = false;                // the variants' states follow from their instances' (wv.inst_state)
    bool steps_stale = false;                    // this table's ix.step_worker is older than its index or the workers
    unsigned long long refreshed_in = 0;         // a capture that has recorded, behind the latest report, what brings these up to date; 0: none
    unsigned long long reported_in = 0;          // the latest capture to record a report, if it has recorded no refresh behind it; 0: none
    bool replays = false;                        // an earlier one did so too: its graph may be replayed in front of any call

    // staircase index
    IndexView ix{};
    bool have_index = false;
    uint32_t index_lds_bytes = 0;     // dynamic LDS of the lookup kernel; 0 = no mirror: every lookup reads lines from global memory
    uint32_t ix_stats[kCtlWords] = {0};      // copy of ix.ctrl taken after the build at load time
    int64_t ix_bytes = 0, ix_steps = 0;      // pool bytes and steps of the index when it was loaded
    int32_t *d_park = nullptr;        // queues of parked queries of the lookup kernel (fixed size)
    int64_t park_bytes = 0;
    uint32_t *host_stats = nullptr;   // pinned, device-visible: six counters of the latest index build (kCtlMaxK0 .., pool, steps)
    int32_t *static_park = nullptr;   // the same queues inside the library's static device array (may be null)
    const uint32_t *last_stats = nullptr;   // statistics of the most recent lookup launch (this table's or the Inactive tier's)
    int32_t last_route = 0;                 // INFAAS_SEL_ROUTE_* of that launch

    // scan scratch
    ScanScratch sc{};
    int64_t sc_capacity = 0;
    int32_t sc_slices = 0;
    int64_t scratch_bytes = 0;
    bool cnt_dirty = false;

    // timing
    bool timing = false;
    std::vector<TimedLaunch> pending;
    std::vector<hipEvent_t> free_events;
    infaas_sel_timings acc{};

    void free_table()
    {
        (void)hipFree(d_acc); (void)hipFree(d_queue); (void)hipFree(d_orig); (void)hipFree(d_lat);
        (void)hipFree(d_rank); (void)hipFree(d_perm); (void)hipFree(d_seg_off);
        (void)hipFree(d_seg_len); (void)hipFree(d_slot_of);
        (void)hipFree(d_acc_r); (void)hipFree(d_orig_r); (void)hipFree(d_row_entry);
        (void)hipFree(d_tot_r);
        d_acc = d_queue = d_orig = d_lat = d_seg_off = d_seg_len = d_slot_of = nullptr;
        d_acc_r = d_orig_r = nullptr;
        d_row_entry = nullptr;
        d_tot_r = nullptr;
        d_rank = d_perm = nullptr;
        (void)hipFree(d_state);
        d_state = nullptr;
        loaded = false;
        reported_in = 0;   // (graphs of the old table's reports are of no use any more)
        replays = false;
        table_bytes = 0;
        for (void *p : scale_mem) (void)hipFree(p);
        scale_mem.clear();
        sv = ScaleView{};
        scaling_loaded = false;
        free_index();
        drop_inactive();
    }
    void drop_inactive();
    void free_index()
    {
        (void)hipFree(ix.pool); (void)hipFree(ix.step_row); (void)hipFree(ix.ctrl);  // hdr lives in pool's allocation
        if (ix.stats) (void)hipFree(ix.stats - 4);
        (void)hipFree(ix.slice_room);   // (rank_hdr and the nodes behind it are in pool's allocation)
        tv.rank_hdr = nullptr;
        (void)hipFree((void *)ix.task_group); (void)hipFree(ix.gctrl);
        (void)hipFree(ix.step_worker); (void)hipFree(ix.hot_worker);
        (void)hipFree(d_park);
        d_park = nullptr;
        park_bytes = 0;
        ix = IndexView{};
        last_stats = nullptr;
        have_index = false;
        index_lds_bytes = 0;
    }
    void free_scratch()
    {
        (void)hipFree(sc.cnt); (void)hipFree(sc.bucket_off); (void)hipFree(sc.cursor);
        (void)hipFree(sc.tile_off); (void)hipFree(sc.wide_off); (void)hipFree(sc.counters);
        (void)hipFree(sc.recs); (void)hipFree(sc.best);
        sc = ScanScratch{};
        sc_capacity = 0;
        sc_slices = 0;
        scratch_bytes = 0;
    }
};

void infaas_sel::drop_inactive()
{
    for (void *p : worker_mem) (void)hipFree(p);
    worker_mem.clear();
    wv = WorkerView{};
    workers_loaded = workers_dirty = rows_stale = instance_states = false;
    (void)hipFree(ix.step_worker); (void)hipFree(ix.hot_worker);
    ix.step_worker = nullptr;
    ix.hot_worker = nullptr;
    (void)hipFree(d_open); (void)hipFree(d_open_count);
    d_open = d_open_count = nullptr;
    open_queries = open_bytes = open_words = 0;
    open_side = false;
    if (inactive) infaas_sel_destroy(inactive);
    inactive = nullptr;
    last_stats = nullptr;
}

namespace {

bool get_event(infaas_sel *h, hipEvent_t *e)
{
    if (!h->free_events.empty()) {
        *e = h->free_events.back();
        h->free_events.pop_back();
        return true;
    }
    return hipEventCreate(e) == hipSuccess;
}

// Hands a launcher the pair of events to attach to its kernel when timing is on.
struct LaunchTimer {
    infaas_sel *h;
    TimedLaunch tl{};
    LaunchEvents pair{};
    bool active = false;
    LaunchTimer(infaas_sel *h_, int kid, hipStream_t) : h(h_)
    {
        if (!h->timing) return;
        tl.kid = kid;
        if (!get_event(h, &tl.a)) return;
        if (!get_event(h, &tl.b)) { h->free_events.push_back(tl.a); return; }
        pair = LaunchEvents{tl.a, tl.b};
        active = true;
    }
    const LaunchEvents *ev() const { return active ? &pair : nullptr; }
    void failed()   // the launch did not happen: the events were never recorded
    {
        if (active) { h->free_events.push_back(tl.a); h->free_events.push_back(tl.b); }
        active = false;
    }
    ~LaunchTimer()
    {
        if (active) h->pending.push_back(tl);
    }
};

int ensure_scratch(infaas_sel *h, int64_t capacity)
{
    const int32_t S = h->T * h->B;
    if (h->sc.recs && h->sc_capacity >= capacity && h->sc_slices == S) return INFAAS_SEL_OK;
    // growing: nothing enqueued earlier may still use the old buffers
    if (!HIP_OK(hipDeviceSynchronize())) return INFAAS_SEL_ERR_HIP;
    int64_t cap = std::max<int64_t>(capacity, h->sc_capacity);
    h->free_scratch();
    ScanScratch sc{};
    bool ok = dev_alloc(&sc.cnt, S) == hipSuccess && dev_alloc(&sc.bucket_off, S + 1) == hipSuccess &&
              dev_alloc(&sc.cursor, S) == hipSuccess && dev_alloc(&sc.tile_off, S + 1) == hipSuccess &&
              dev_alloc(&sc.wide_off, S + 1) == hipSuccess && dev_alloc(&sc.counters, 4) == hipSuccess &&
              dev_alloc(&sc.recs, (size_t)cap) == hipSuccess && dev_alloc(&sc.best, (size_t)cap) == hipSuccess;
    h->sc = sc;
    if (!ok) {
        h->free_scratch();
        (void)hipGetLastError();
        return INFAAS_SEL_ERR_OOM;
    }
    if (!HIP_OK(hipMemset(sc.cnt, 0, std::max<size_t>(S, 1) * 4)) ||
        !HIP_OK(hipMemset(sc.counters, 0, 16))) {
        h->free_scratch();
        return INFAAS_SEL_ERR_HIP;
    }
    h->cnt_dirty = false;
    h->sc_capacity = cap;
    h->sc_slices = S;
    h->scratch_bytes = (int64_t)S * 4 * 5 + 8 + 16 + cap * (16 + 4);
    return INFAAS_SEL_OK;
}

constexpr uint32_t kLdsMax = 160 * 1024;  // dynamic LDS the lookup kernel may ask for

// Groups of tasks (IndexView::num_groups).  What they are for is the spread of the build's requests for room over as many pairs of
// counters; any sizes that make tens of groups of a table with thousands of slices do.
constexpr uint32_t kGroupRegionBytes = 144 * 1024;   // bytes of a group's bodies
constexpr uint32_t kGroupMaxSlices = 1900;
constexpr uint32_t kGroupStepCap = 16384;            // entries of step_row per group (a region holds at most 10,532 steps)
constexpr int32_t kGroupMaxGroups = 120;
constexpr int32_t kGroupMaxTasks = 16384;            // of a table in groups; one of more tasks keeps one region
constexpr uint32_t kGroupHotRows = 8;

// Starting values of the allocator counters and the statistics, then one build, then the counters back.
int build_index_now(infaas_sel *h)
{
    IndexView &ix = h->ix;
    const bool grouped = ix.num_groups > 1;
    uint32_t ctrl0[kCtlWords] = {0};
    ctrl0[kCtlPool] = ctrl0[kCtlPool0] = grouped ? ix.num_groups * ix.region_bytes : kDummyBodyBytes;
    ctrl0[kCtlSteps] = ctrl0[kCtlSteps0] = grouped ? ix.num_groups * ix.group_step_cap : 1u;
    ctrl0[kCtlMaxK0] = 1u;
    ctrl0[kCtlEpoch] = 1u;   // (slice_room is cleared below: build number 0)
    std::vector<uint32_t> g0;
    for (uint32_t g = 0; grouped && g < ix.num_groups; ++g) { g0.push_back(kDummyBodyBytes); g0.push_back(g == 0 ? 1u : 0u); }
    if (!HIP_OK(hipMemcpy(ix.ctrl, ctrl0, sizeof(ctrl0), hipMemcpyHostToDevice)) ||
        !HIP_OK(hipMemset(ix.slice_room, 0, (size_t)h->T * h->B * sizeof(unsigned long long))) ||
        (grouped && !HIP_OK(hipMemcpy(ix.gctrl, g0.data(), g0.size() * 4, hipMemcpyHostToDevice))) ||
        !HIP_OK(launch_index_build(h->tv, ix, nullptr)) || !HIP_OK(hipDeviceSynchronize()) ||
        !HIP_OK(hipMemcpy(h->ix_stats, ix.ctrl, sizeof(ctrl0), hipMemcpyDeviceToHost)))
        return INFAAS_SEL_ERR_HIP;
    // what the selections' first kernels keep up to date from now on
    if (h->host_stats) {
        void *dev = nullptr;
        for (int i = 0; i < 4; ++i) h->host_stats[i] = h->ix_stats[kCtlMaxK0 + i];
        h->host_stats[4] = h->ix_stats[kCtlPool];
        h->host_stats[5] = h->ix_stats[kCtlSteps];
        if (hipHostGetDevicePointer(&dev, h->host_stats, 0) == hipSuccess) {
            h->tv.stat_src = ix.ctrl;
            h->tv.stat_dst = (uint32_t *)dev;
        } else {
            (void)hipGetLastError();
        }
    }
    // bytes and steps of the index as a whole (info only)
    h->ix_bytes = h->ix_stats[kCtlPool];
    h->ix_steps = (int64_t)h->ix_stats[kCtlSteps] - 1;   // (entry 0 of step_row is unused)
    if (grouped) {
        if (!HIP_OK(hipMemcpy(g0.data(), ix.gctrl, g0.size() * 4, hipMemcpyDeviceToHost))) return INFAAS_SEL_ERR_HIP;
        h->ix_bytes -= (int64_t)ix.num_groups * ix.region_bytes;
        h->ix_steps -= (int64_t)ix.num_groups * ix.group_step_cap;
        for (uint32_t g = 0; g < ix.num_groups; ++g) { h->ix_bytes += g0[2 * g]; h->ix_steps += g0[2 * g + 1]; }
    }
    return INFAAS_SEL_OK;
}

// Allocate the staircase index for the loaded table, build it and read its sizes back.
int create_index(infaas_sel *h)
{
    const int64_t S = (int64_t)h->T * h->B;
    const uint32_t worst = 2 * body_bytes(body_re(kBodySteps)) + 2 * (kBodySteps + 1);
    // The build takes room with one add on a pair of 32-bit counters; their sums must not carry.
    // A table with that many slices (millions) gets no index and is answered by the scan engine.
    const int64_t regions = (int64_t)kGroupMaxGroups * kGroupRegionBytes, region_steps = (int64_t)kGroupMaxGroups * kGroupStepCap;
    if (regions + kDummyBodyBytes + S * worst > 0xFFFF0000ll || region_steps + 1 + S * kIndexCap > 0xFFFF0000ll) return INFAAS_SEL_OK;
    IndexView ix{};
    ix.num_groups = 1;
    // room for the regions of a grouped layout in front of what an ungrouped one needs
    ix.pool_bytes = (uint32_t)std::min<int64_t>(regions + kDummyBodyBytes + S * worst + 64, (int64_t)3 << 30);
    ix.step_cap = (uint32_t)std::min<int64_t>(region_steps + 1 + S * kIndexCap, (int64_t)1 << 29);
    // the header of an empty slice, and the slices as the search in rank order sees them (TableView::rank_hdr)
    std::vector<uint32_t> hdrs{0u, kEmptyHdrY, 0u, 4u + body_bytes(2)};
    hdrs.resize(4 + ((size_t)S + 1) * 4, 0u);
    int64_t nodes = 0;
    {
        std::vector<int32_t> len((size_t)h->T, 0);
        for (int32_t t : h->h_task) len[(size_t)t] += 1;
        int64_t seg = 0;
        for (int32_t t = 0; t < h->T; ++t) {
            const int32_t L = len[(size_t)t], n = all_level_nodes(L) + rank_blocks(L) * kRankBlockNodes;
            for (int32_t b = 0; b < h->B; ++b, nodes += n) {
                uint32_t *e = &hdrs[4 + ((size_t)t * h->B + b) * 4];
                e[0] = (uint32_t)(((int64_t)b * h->Vp + seg) / 4); e[1] = (uint32_t)L; e[2] = (uint32_t)nodes;
            }
            seg += (L + 3) & ~3;
        }
    }
    // keys run from 1 to the highest accuracy's (as far as there are keys for it), thresholds to one more
    int64_t top = 1;
    for (int32_t a : h->h_acc) top = std::max<int64_t>(top, std::min<int64_t>((int64_t)a - h->tv.acc_base, 65533) + 1);
    ix.line_form = std::min(kLineMaxShift, (uint32_t)__builtin_clz((uint32_t)(top + 1)));
    ix.line_top = (uint32_t)top + 1u;
    if (h->V > (int64_t)1 << ix.line_shift()) ix.line_form |= 1u << 31;
    // one allocation: the pool, then the headers, so that one 32-bit offset reaches both; behind them rank_hdr and,
    // at a multiple of their size, the nodes of TableView::rank_nodes and the lines (counted with the table: they do not follow the index)
    ix.pool_bytes &= ~127u;
    const size_t nstats = (size_t)index_stat_blocks(h->num_cus) * kLookupStats;
    bool ok = dev_alloc(&ix.pool, (size_t)ix.pool_bytes + rank_nodes_at((int32_t)S) + (size_t)std::max<int64_t>(nodes, 1) * 128 + (size_t)kLinePlanes * line_plane((int32_t)S)) == hipSuccess &&
              dev_alloc(&ix.step_row, ix.step_cap) == hipSuccess && dev_alloc(&ix.ctrl, kCtlWords) == hipSuccess &&
              dev_alloc(&ix.stats, 4 + nstats) == hipSuccess && dev_alloc(&ix.gctrl, 2 * (size_t)kGroupMaxGroups) == hipSuccess &&
              dev_alloc(&ix.slice_room, (size_t)S) == hipSuccess;
    if (ix.stats) ix.stats += 4;   // (in front of it how many entries are in use)
    if (ok) {
        ix.hdr = (uint4 *)(ix.pool + ix.pool_bytes);
        ix.lines = (uint8_t *)ix.hdr + rank_nodes_at((int32_t)S) + (size_t)std::max<int64_t>(nodes, 1) * 128;
        h->tv.rank_hdr = (const uint4 *)((char *)ix.hdr + rank_hdr_at((int32_t)S));
    }
    h->ix = ix;
    const size_t park = index_park_bytes(h->num_cus);
    ok = ok && dev_alloc(&h->d_park, park / 4) == hipSuccess;
    h->park_bytes = ok ? (int64_t)park : 0;
    if (!ok) {
        h->free_index();
        (void)hipGetLastError();
        return INFAAS_SEL_ERR_OOM;
    }
    // dummy body of a slice without steps (sentinels only) at offset 0; step_row[0] is never an answer
    uint8_t dummy[kDummyBodyBytes] = {0};
    for (uint32_t i = 8; i < 16; ++i) dummy[i] = 0xFF;  // latency sentinels of the empty body (Re = 2)
    const int32_t none = -1;
    uint2 empty[kLineBytes / 8];   // the line of the empty slice
    for (uint2 &e : empty) e = make_uint2(0u, kLineEnd);
    if (!HIP_OK(hipMemset(ix.stats - 1, 0, 4)) ||
        !HIP_OK(hipMemcpy(ix.lines + (size_t)S * kLineBytes, empty, sizeof(empty), hipMemcpyHostToDevice)) ||
        !HIP_OK(hipMemcpy(ix.pool, dummy, sizeof(dummy), hipMemcpyHostToDevice)) ||
        !HIP_OK(hipMemcpy(ix.step_row, &none, 4, hipMemcpyHostToDevice)) ||
        !HIP_OK(hipMemcpy(&ix.hdr[S], hdrs.data(), hdrs.size() * 4, hipMemcpyHostToDevice)) ||
        build_index_now(h) != INFAAS_SEL_OK) {
        h->free_index();
        return INFAAS_SEL_ERR_HIP;
    }
    h->have_index = true;
    h->table_bytes += (S + 1) * 16 + nodes * 128 + (S + 1) * kLinePlanes * kLineBytes;
    const int64_t fixed = kLdsCtrlBytes + lds_header_bytes((int32_t)S) + 16;
    const int64_t need = fixed + h->ix_stats[kCtlPool];
    // The lookup kernel mirrors the index in LDS when the slice headers leave at least half of it to
    // the bodies; bodies that do not fit stay in global memory and their queries take the slower
    // path inside the same kernel.  With more headers than that there is no mirror (memory_pays()).
    h->index_lds_bytes = fixed <= (int64_t)kLdsMax / 2 ? kLdsMax : 0u;
    // 2 bytes of a step's caller row sit in front of its body, the bits above in a 14-bit header field
    const uint32_t row_bits = h->V > 1 ? 64u - (uint32_t)__builtin_clzll((unsigned long long)(h->V - 1)) : 1u;
    h->ix.row_hi_bits = row_bits > 16 ? row_bits - 16 : 0u;
    const uint32_t hot_max = std::min<uint32_t>(h->ix.row_hi_bits ? kRowHiField / h->ix.row_hi_bits : (uint32_t)kBodySteps, kBodySteps);
    if (need > 2 * (int64_t)kLdsMax && h->T <= kGroupMaxTasks) {
        // Not even half of the bodies fit one LDS, so mostly thousands of slices: deal the tasks, in order, to groups whose
        // bodies fit a region (with a fifth of it left free, because staircases grow and shrink with the load), and build
        // again with one region of the pool per group, each with its own allocation counters: the slices
        // do not wait for their turn at one pair.
        std::vector<uint32_t> hdr((size_t)S * 4);
        if (!HIP_OK(hipMemcpy(hdr.data(), h->ix.hdr, (size_t)S * 16, hipMemcpyDeviceToHost))) { h->free_index(); return INFAAS_SEL_ERR_HIP; }
        const uint32_t hot = std::min(kGroupHotRows, hot_max) & ~1u;
        const uint32_t target = (kGroupRegionBytes - kDummyBodyBytes) / 5 * 4;
        std::vector<uint16_t> task_group((size_t)h->T);
        int32_t G = 1;
        uint32_t bytes = 0, slices = 0;
        for (int32_t t = 0; t < h->T; ++t) {
            uint32_t tb = 0;
            for (int32_t b = 0; b < h->B; ++b) {
                const uint32_t *e = &hdr[((size_t)t * h->B + b) * 4];   // {body address, y, first step, end of bodies}
                if (e[0] != 0u) tb += e[3] - (e[0] + 4u) + 2u * hot + 4u;   // bodies, and room for the first steps' rows
            }
            if (slices > 0 && (bytes + tb > target || slices + (uint32_t)h->B > kGroupMaxSlices)) {
                ++G;
                bytes = slices = 0;
            }
            bytes += tb; slices += (uint32_t)h->B;
            task_group[(size_t)t] = (uint16_t)(G - 1);
        }
        if (G > 1 && G <= kGroupMaxGroups && (uint32_t)h->B <= kGroupMaxSlices) {
            uint16_t *d_tg = nullptr;
            if (dev_alloc(&d_tg, (size_t)h->T) != hipSuccess) {
                (void)hipGetLastError();
                h->free_index();
                return INFAAS_SEL_ERR_OOM;
            }
            h->ix.task_group = d_tg;
            h->ix.num_groups = (uint32_t)G; h->ix.region_bytes = kGroupRegionBytes; h->ix.group_step_cap = kGroupStepCap;
            h->ix.hot_rows = hot;
            bool up = HIP_OK(hipMemcpy(d_tg, task_group.data(), (size_t)h->T * 2, hipMemcpyHostToDevice));
            for (int32_t g = 1; up && g < G; ++g)   // every region begins with the dummy body
                up = HIP_OK(hipMemcpy(h->ix.pool + (size_t)g * kGroupRegionBytes, dummy, sizeof(dummy), hipMemcpyHostToDevice));
            if (!up || build_index_now(h) != INFAAS_SEL_OK) { h->free_index(); return INFAAS_SEL_ERR_HIP; }
            return INFAAS_SEL_OK;
        }
    }
    // LDS left over holds the caller rows of the first steps of every slice (the steps most answers
    // come from), which saves those answers a gather from global memory.  Rebuild with that many.
    const int64_t spare = (int64_t)kLdsMax - need - 1024;   // keep room for staircases that grow with load
    const uint32_t hot = spare > 0 ? (uint32_t)std::min<int64_t>((spare / (4 * S)) * 2, hot_max) : 0u;
    if (h->index_lds_bytes && hot > 0) {
        h->ix.hot_rows = hot;
        if (build_index_now(h) != INFAAS_SEL_OK) {
            h->free_index();
            return INFAAS_SEL_ERR_HIP;
        }
    }
    return INFAAS_SEL_OK;
}

// Lists for the queries that the first tier of a state-aware pass over up to n queries leaves open.
// side: also the lists of the first tier's suggestions beside them (complete Case I), the same size again.
bool open_there(const infaas_sel *h, int64_t n, bool side)
{
    return h->d_open && h->open_queries >= n && (h->open_side || !side);
}
int ensure_open(infaas_sel *h, int64_t n, bool side)
{
    if (open_there(h, n, side)) return INFAAS_SEL_OK;
    n = std::max(n, h->open_queries);
    side = side || h->open_side;
    // growing: nothing enqueued earlier may still use the old lists
    if (!HIP_OK(hipDeviceSynchronize())) return INFAAS_SEL_ERR_HIP;
    (void)hipFree(h->d_open);
    h->d_open = nullptr;
    h->open_queries = h->open_bytes = 0;
    const int blocks = index_select_blocks(h->num_cus);
    h->open_side = false;
    const size_t words = (size_t)blocks * (size_t)index_open_cap((int32_t)n, h->num_cus) * 4;
    if (!h->d_open_count && dev_alloc(&h->d_open_count, (size_t)blocks) != hipSuccess) return INFAAS_SEL_ERR_OOM;
    if (dev_alloc(&h->d_open, words * (side ? 2 : 1)) != hipSuccess) return INFAAS_SEL_ERR_OOM;
    h->open_queries = n;
    h->open_words = (int64_t)words;
    h->open_side = side;
    h->open_bytes = (int64_t)words * 4 * (side ? 2 : 1);
    return INFAAS_SEL_OK;
}

// Bytes of the bodies of the index as of its latest build that is known of (in groups: when it was loaded).
int64_t body_pool(const infaas_sel *h)
{
    const volatile uint32_t *now = h->host_stats;
    return h->ix.num_groups > 1 ? h->ix_bytes : now ? now[4] : h->ix_stats[kCtlPool];
}

// Which way a lookup goes.  The mirror costs its fill (2-4 us, more with many slices) and pays with 4 ps per query, if it holds the
// query's slice and the slice's first body has the answer; a line read from memory costs 7 to 9, one query per lane or, with a tile of them
// at a time, 6 to 8 and a start of 2 us.
struct IndexShape {
    int64_t pool, room;   // bytes of the bodies, and what the mirror has for them (0: no mirror)
    double outside;       // share of the bodies outside the mirror
    double open;          // share of the slices that the index does not hold completely
    double steps;         // per slice
    uint32_t most;        // steps of the slice that has most
};
IndexShape shape_of(const infaas_sel *h)
{
    const volatile uint32_t *now = h->host_stats;
    const bool fresh = now && h->ix.num_groups <= 1;
    const double S = std::max(1, h->T * h->B);
    IndexShape x{};
    x.pool = body_pool(h);
    x.room = h->index_lds_bytes == 0 ? 0 : (int64_t)h->index_lds_bytes - kLdsCtrlBytes - lds_header_bytes(h->tv.S);
    x.outside = x.pool > x.room ? 1.0 - (double)x.room / (double)x.pool : 0.0;
    x.open = (now ? now[kCtlTrunc - kCtlMaxK0] + now[kCtlNoBody - kCtlMaxK0] : h->ix_stats[kCtlTrunc] + h->ix_stats[kCtlNoBody]) / S;
    x.steps = (fresh ? (double)now[5] : (double)h->ix_steps) / S;
    x.most = now ? now[kCtlMaxK - kCtlMaxK0] : h->ix_stats[kCtlMaxK];
    return x;
}
// The plain selection: whether the mirror is ahead of the lines from `n` queries on.  us for 300,000 / 600,000 / 1M / 4M / 16M queries, a lane
// per query (a tile at a time) and mirrored: 50 tasks of 2000 variants, all in the mirror, 7.0 / 11.2 / 16.0 / 50 / 209 (-, -, 14.9 / 42 / 151)
// and 8.2 / 10.1 / 11.3 / 25 / 72; 100 of 200, 8% outside, 6.5 / 10.4 / 14.4 / 45 / 196 (-, -, 13.5 / 40 / 146) and 9.7 / 12.0 / 14.3 / 39 / 142; 200 of 60,
// half outside, 6.2 / 9.5 / 13.1 / 39 / 180 (-, -, 13.0 / 38 / 135) and 13.2 / 17.7 / 24.0 / 73 / 279.  So a query pays 50 ps for every share
// of the bodies outside, 4.7 less than from a line otherwise, and the start 1.5 us more; slices that are not completely indexed, which the
// lookup kernel scans, cost 2.3 ns.
bool mirror_pays(const IndexShape &x, int64_t n)
{
    return x.room > 0 && n > 350000 && 50.0 * x.outside + 2300.0 * x.open + 1.5e6 / (double)n < 4.7;
}
// ... and where it is not, from how many queries on a tile at a time is ahead of a lane per query.  us, a lane per query / a tile at a time, for
// 600,000 / 900,000 / 1.3M / 1.6M / 2.5M / 5M queries, arrays of up to three calls (of 5M no more) in the last-level cache: 1000 tasks of 100
// variants on average 10.3 / 12.6, 12.4 / 14.1, 16.2 / 17.7, 18.9 / 19.1, 25.7 / 26.7, 60 / 46; 400 of 60 9.3 / 10.8, 11.9 / 12.6, 15.6 / 16.3, 18.3 / 17.6, 25.0 /
// 24.9, 58 / 44; 100 of 200 8.7 / 10.6, 11.3 / 12.1, 15.4 / 15.9, 18.2 / 17.2, 24.3 / 24.5, 55 / 46; 2000 of 20 8.4 / 9.9, 9.9 / 11.4, 12.9 / 15.8, 15.2 / 16.5, 20.3 /
// 25.0, 48 / 43.  (64M queries on 8000 slices, binned by group of tasks whose bodies fit one LDS, 684, so 453.)
constexpr int64_t kTileQueries = 1500000;
// With suggestions (b null), and in two tiers (a the Active one, which all queries visit), whether a lane per query straight from memory is
// ahead of the mirror.  Both are a start and a time per query, here in us and us per million; the crossing moves with the steps per slice (fewer
// steps: more queries without an answer, each of them a drain and a second tier for the mirror), with the share of the bodies outside and
// with the slices that are not completely indexed (2.3 ns per query in the lookup kernel's scan).  us, memory / mirror:
//   tasks x variants x batches  steps  outside                 300,000        600,000        1M             1.5M           2.2M           4M
//   suggestions
//     8 x 32 x 4                   9   0                         8.3 / 10.4                   18.1 / 13.7    23.3 / 19.3                   (450,000: 9.9 / 11.1)
//     40 x 100 x 8                11   0                        10.2 / 10.6                   23.2 / 14.0    30.7 / 19.4                   (450,000: 12.3 / 11.1)
//     50 x 2000 x 8               24   0                        12.0 / 11.0                   26.6 / 14.0    35.5 / 16.9                   (200,000: 8.8 / 10.6)
//     200 x 400 x 3               18   0.05                     11.0 / 13.5                   24.2 / 19.1    32.4 / 26.4                   (450,000: 13.2 / 14.5)
//     100 x 200 x 8               14   0.11                     10.2 / 15.2                   23.6 / 21.4    30.7 / 29.3                   (700,000: 17.7 / 18.6)
//     100 x 600 x 8               20   0.34                     11.3 / 20.1                   25.3 / 30.7    33.6 / 40.0                   (5M: 110 / 101)
//     200 x 60 x 8                10   0.40                     10.5 / 24.6                   23.3 / 36.2    31.4 / 50.0                   (16M: 305 / 383)
//   two tiers, behind a state report
//     40 x 100 x 8                 9   0                        23.3 / 30.8    27.9 / 33.3    33.1 / 36.0    38.9 / 40.5    47.9 / 47.0    80 / 61
//     50 x 2000 x 8               20   0                        30.4 / 37.8    34.5 / 39.1    39.5 / 40.6    45.4 / 44.2    55.3 / 49.0    90 / 60
//     100 x 600 x 8               16   0.19                     30.4 / 40.5    34.3 / 42.8    39.2 / 46.9    44.8 / 53.8    54.5 / 62.0    89 / 82
//     200 x 60 x 8                 7   0.23                     26.0 / 34.4    30.3 / 41.3    34.9 / 45.7    40.8 / 52.9    49.8 / 62.4    83 / 90
//   with workers, behind reports on them and on instance states
//     40 x 100 x 8                 9   0                        30.1 / 40.7                   40.8 / 47.1    46.5 / 52.2                   96 / 78
//     50 x 2000 x 8               21   0                        40.9 / 50.0                   50.5 / 53.6    56.8 / 58.2                   110 / 78
//   complete Case I, with workers
//     8 x 32 x 4                   6   0                        15.5 / 33.3    23.9 / 37.7    34.6 / 41.3    45.1 / 51.4    65.8 / 67.5    125 / 109
//     100 x 200 x 8               11   0                        16.3 / 33.2    25.1 / 37.7    36.0 / 42.5    47.2 / 49.7    68.4 / 62.6    129 / 105
//     50 x 2000 x 8               20   0                        16.9 / 24.2    26.2 / 29.9    37.8 / 34.1    50.5 / 39.9    71.1 / 45.0    133 / 64
//     100 x 600 x 8               16   0.20                     17.1 / 37.6    26.1 / 46.1    37.7 / 52.1    49.3 / 62.9    71.4 / 75.8    135 / 119
//     200 x 60 x 8                 7   0.23                     17.1 / 49.3    25.8 / 54.3    36.6 / 61.3    48.7 / 81.9    69.2 / 114     130 / 183
// Without a mirror (16,000 slices) there is only the way from memory; a lookup kernel that read the bodies from there took two to four times as long
// (suggestions for 349,999 / 4M queries 29 and 269 against 12 and 75, two tiers 2M 224 against 129).
bool memory_pays(const IndexShape &a, const IndexShape *b, bool workers, bool closest, int64_t n)
{
    if (a.room == 0 || (b && b->room == 0)) return true;
    const double m = 1e-6 * (double)n, steps = a.steps, outside = a.outside + (b ? b->outside : 0.0);
    double memory, start, each;   // the mirror's: start + each * m
    if (!b) {
        memory = 5.0 + (a.most < 16u ? 14.0 : 17.5 + 0.14 * steps) * m;   // (below 16 steps no slice has a second line)
        start = outside > 0 ? 10.8 + 15.0 * outside : 9.3;
        each = outside > 0 ? 7.5 + 27.0 * outside : 4.7;
    } else if (closest) {
        memory = 7.5 + 28.2 * m + 3.5 * std::max(0.0, m - 2.2);   // (beyond, the last-level cache does not hold the arrays of several calls)
        start = std::max(20.0, 32.0 - 0.6 * steps) + 40.0 * outside;
        each = std::max(9.0, 21.0 - 0.5 * steps) + 700.0 / std::max(1.0, steps) * outside;
    } else {
        memory = (workers ? 13.4 : 13.2) * m + 5.5 * std::max(0.0, m - 2.5);
        start = workers ? 10.6 : 9.0;
        each = std::max(5.5, (workers ? 10.8 : 9.8) - 0.19 * steps) + 25.0 * outside;
    }
    each += 2300.0 * (a.open + (b ? b->open : 0.0));
    return memory <= start + each * m;
}

// The plain selection, n <= 2^28 queries.  park: the lookup kernel's queues.
hipError_t launch_select(infaas_sel *h, const QueryView &q, int32_t *park, hipStream_t st, const LaunchEvents *ev = nullptr)
{
    const IndexShape x = shape_of(h);
    h->last_route = mirror_pays(x, q.n) ? INFAAS_SEL_ROUTE_MIRROR : q.n >= kTileQueries ? INFAAS_SEL_ROUTE_TILES : INFAAS_SEL_ROUTE_MEMORY;
    if (h->last_route == INFAAS_SEL_ROUTE_MIRROR) return launch_index_select(h->tv, h->ix, q, park, h->index_lds_bytes, h->num_cus, st, ev);
    if (h->last_route == INFAAS_SEL_ROUTE_TILES) return launch_line_select(h->tv, h->ix, q, h->num_cus, st, ev);
    return launch_direct_select(h->tv, h->ix, q, false, h->num_cus, st, ev);
}

// One pass of the index engine over n <= 2^28 queries.
int index_pass(infaas_sel *h, const QueryView &q, hipStream_t st)
{
    LaunchTimer t(h, INFAAS_SEL_K_INDEX_SELECT, st);
    if (q.pass == 0) return HIP_OK(launch_select(h, q, h->d_park, st, t.ev())) ? INFAAS_SEL_OK : INFAAS_SEL_ERR_HIP;
    if (q.pass == 1) {
        const IndexShape x = shape_of(h);
        if (memory_pays(x, nullptr, false, true, q.n)) {
            h->last_route = INFAAS_SEL_ROUTE_MEMORY;
            const hipError_t e = launch_direct_modes(h->tv, h->ix, h->tv, h->ix, q, false, x.open > 0, h->num_cus, st, t.ev());
            return HIP_OK(e) ? INFAAS_SEL_OK : INFAAS_SEL_ERR_HIP;
        }
    }
    h->last_route = INFAAS_SEL_ROUTE_MIRROR;
    if (!HIP_OK(launch_index_select(h->tv, h->ix, q, h->d_park, h->index_lds_bytes, h->num_cus, st, t.ev())))
        return INFAAS_SEL_ERR_HIP;
    return INFAAS_SEL_OK;
}

bool use_index(infaas_sel *h)
{
    const uint32_t engine = h->flags & INFAAS_SEL_ENGINE_MASK;
    if (!h->have_index || engine == INFAAS_SEL_ENGINE_SCAN) return false;
    if (engine == INFAAS_SEL_ENGINE_INDEX) return true;
    // The first kernel of every selection copies four counters of the latest index build into pinned
    // host memory (TableView::stat_dst), so what is read here is at most one call behind, and no
    // call ever waits for it.
    uint32_t trunc = h->ix_stats[kCtlTrunc], nobody = h->ix_stats[kCtlNoBody];
    if (h->host_stats) {
        trunc = ((volatile uint32_t *)h->host_stats)[kCtlTrunc - kCtlMaxK0];
        nobody = ((volatile uint32_t *)h->host_stats)[kCtlNoBody - kCtlMaxK0];
    }
    // auto: the index, unless
    // more than half of the slices could not be indexed completely when the table was loaded or, as
    // far as is known by now, when the index was last rebuilt -- their queries would mostly end in
    // the in-kernel scan, and use_ranked()'s search or, without it, the bucketed scan engine does
    // those faster.  (The share was chosen for that engine.  By the search's figures it pays from
    // a few hundredths of the queries on: one that the lookup kernel scans for costs 2.3 ns there and 0.04 ns in rank order,
    // one that the mirror answers 0.004 ns.)
    const int64_t S = (int64_t)h->T * h->B;
    return 2 * ((int64_t)trunc + nobody) <= S;
}

// Whether a table that the index engine is not used for is answered in rank order instead of by the exhaustive scan:
// always when there is an index, whose build writes what the search needs.  4M queries on 50 tasks of 2000 variants, the
// scan engine's four kernels against this one: every variant a step 2.80 ms against 0.12, accuracies beyond 16 bits 2.79
// against 0.16, config 2 after the degrading report 2.84 against 0.06, steps in random order 2.80 against 1.39, two
// interleaved families of variants with most queries asking for the best of both 2.77 against 1.21.  Slices of 64 to 20,000
// entries and batches of 101 to 1M queries: faster throughout.
bool use_ranked(const infaas_sel *h)
{
    return h->have_index && (h->flags & INFAAS_SEL_ENGINE_MASK) == INFAAS_SEL_ENGINE_AUTO;
}

// One pass over a table that the index engine is not used for although there is an index (automatic mode): most
// slices are answered from their entries in rank order.
int ranked_pass(infaas_sel *h, const QueryView &q, hipStream_t st)
{
    LaunchTimer t(h, INFAAS_SEL_K_SCAN_LDS, st);
    if (!HIP_OK(launch_direct_select(h->tv, h->ix, q, true, h->num_cus, st, t.ev()))) return INFAAS_SEL_ERR_HIP;
    return INFAAS_SEL_OK;
}

// One pass of the scan engine over n <= 2^28 queries.
int scan_pass(infaas_sel *h, const QueryView &q, hipStream_t st)
{
    if (h->cnt_dirty) {  // an earlier call failed between histogram and plan
        if (!HIP_OK(hipStreamSynchronize(st))) return INFAAS_SEL_ERR_HIP;
        if (!HIP_OK(hipMemset(h->sc.cnt, 0, (size_t)h->tv.S * 4))) return INFAAS_SEL_ERR_HIP;
        h->cnt_dirty = false;
    }
    h->cnt_dirty = true;
    {
        LaunchTimer t(h, INFAAS_SEL_K_HISTOGRAM, st);
        if (!HIP_OK(launch_histogram(h->tv, q, h->sc, st, t.ev()))) return INFAAS_SEL_ERR_HIP;
    }
    {
        LaunchTimer t(h, INFAAS_SEL_K_PLAN, st);
        if (!HIP_OK(launch_plan(h->tv, h->sc, st, t.ev()))) return INFAAS_SEL_ERR_HIP;
    }
    h->cnt_dirty = false;
    const bool wide = h->wide_segments > 0;
    {
        LaunchTimer t(h, INFAAS_SEL_K_SCATTER, st);
        if (!HIP_OK(launch_scatter(h->tv, q, h->sc, wide, st, t.ev()))) return INFAAS_SEL_ERR_HIP;
    }
    if (h->max_lds_segment > 0) {
        LaunchTimer t(h, INFAAS_SEL_K_SCAN_LDS, st);
        if (!HIP_OK(launch_scan_lds(h->tv, q, h->sc, h->max_lds_segment, h->num_cus, st, t.ev())))
            return INFAAS_SEL_ERR_HIP;
    }
    if (wide) {
        {
            LaunchTimer t(h, INFAAS_SEL_K_SCAN_WIDE, st);
            if (!HIP_OK(launch_scan_wide(h->tv, q, h->sc, h->num_cus, st, t.ev())))
                return INFAAS_SEL_ERR_HIP;
        }
        LaunchTimer t(h, INFAAS_SEL_K_FINISH_WIDE, st);
        if (!HIP_OK(launch_finish_wide(h->tv, q, h->sc, st, t.ev()))) return INFAAS_SEL_ERR_HIP;
    }
    return INFAAS_SEL_OK;
}

constexpr int64_t kMaxPass = (int64_t)1 << 28;
// State-aware selection: 16 bytes of list memory per query of a pass, hence shorter passes.
constexpr int64_t kMaxTierPass = (int64_t)1 << 26;

}  // namespace

extern "C" {

const char *infaas_sel_last_error(void) { return g_last_error; }

const char *infaas_sel_strerror(int status)
{
    switch (status) {
    case INFAAS_SEL_OK: return "ok";
    case INFAAS_SEL_ERR_INVALID_ARG: return "invalid argument";
    case INFAAS_SEL_ERR_NOT_LOADED: return "no variant table loaded";
    case INFAAS_SEL_ERR_OUT_OF_RANGE: return "table value out of range";
    case INFAAS_SEL_ERR_HIP: return "HIP runtime error";
    case INFAAS_SEL_ERR_OOM: return "out of memory";
    default: return "unknown status";
    }
}

int infaas_sel_create(const infaas_sel_config *cfg, infaas_sel_t **out)
{
    if (!cfg || !out) return INFAAS_SEL_ERR_INVALID_ARG;
    if (cfg->num_tasks < 1 || cfg->num_batch_sizes < 1 || cfg->num_batch_sizes > 64)
        return INFAAS_SEL_ERR_INVALID_ARG;
    if ((int64_t)cfg->num_tasks * cfg->num_batch_sizes > ((int64_t)1 << 24))
        return INFAAS_SEL_ERR_INVALID_ARG;
    uint32_t engine = cfg->flags & INFAAS_SEL_ENGINE_MASK;
    if ((cfg->flags & ~INFAAS_SEL_ENGINE_MASK) != 0 || engine > INFAAS_SEL_ENGINE_INDEX)
        return INFAAS_SEL_ERR_INVALID_ARG;
    int32_t lim = cfg->lds_segment_limit == 0 ? 4096 : cfg->lds_segment_limit;
    if (lim < 64 || lim > 8192) return INFAAS_SEL_ERR_INVALID_ARG;
    lim &= ~63;
    int ndev = 0;
    if (!HIP_OK(hipGetDeviceCount(&ndev))) return INFAAS_SEL_ERR_HIP;
    if (cfg->device < 0 || cfg->device >= ndev) return INFAAS_SEL_ERR_INVALID_ARG;

    infaas_sel *h = new (std::nothrow) infaas_sel();
    if (!h) return INFAAS_SEL_ERR_OOM;
    h->T = cfg->num_tasks;
    h->B = cfg->num_batch_sizes;
    h->device = cfg->device;
    h->flags = cfg->flags;
    h->lds_limit = lim;
    if (cfg->batch_sizes) h->batch_sizes.assign(cfg->batch_sizes, cfg->batch_sizes + h->B);
    hipDeviceProp_t prop;
    if (!HIP_OK(hipGetDeviceProperties(&prop, h->device))) {
        delete h;
        return INFAAS_SEL_ERR_HIP;
    }
    h->num_cus = prop.multiProcessorCount > 0 ? prop.multiProcessorCount : 256;
    {
        DeviceGuard g(h->device);
        if (g.ok && hipHostMalloc((void **)&h->host_stats, 64, hipHostMallocMapped) != hipSuccess) {
            (void)hipGetLastError();
            h->host_stats = nullptr;
        }
    }
    {
        // address of the static scratch array on this device, for infaas_sel_select_noalloc (a
        // failure here only makes that one call unavailable)
        DeviceGuard g(h->device);
        if (g.ok) h->static_park = (int32_t *)static_scratch(h->device);
    }
    *out = h;
    return INFAAS_SEL_OK;
}

int infaas_sel_load_variants(infaas_sel_t *h, int32_t V, const int32_t *task_id,
                             const int32_t *acc_bp, const int32_t *lat_us, const int32_t *cost,
                             const int32_t *queue_us)
{
    if (!h || V < 0) return INFAAS_SEL_ERR_INVALID_ARG;
    if (V > 0 && (!task_id || !acc_bp || !lat_us || !cost || !queue_us))
        return INFAAS_SEL_ERR_INVALID_ARG;
    const int32_t T = h->T, B = h->B;

    // ---- validate ranges before touching the old table
    for (int64_t v = 0; v < V; ++v) {
        if (task_id[v] < 0 || task_id[v] >= T || queue_us[v] < 0) return INFAAS_SEL_ERR_OUT_OF_RANGE;
        for (int32_t b = 0; b < B; ++b)
            if (lat_us[v * B + b] < 0 || cost[v * B + b] < 0) return INFAAS_SEL_ERR_OUT_OF_RANGE;
    }

    std::vector<int32_t> keep_task(task_id, task_id + V), keep_acc(acc_bp, acc_bp + V),
        keep_lat(lat_us, lat_us + (size_t)V * B);

    // ---- group rows by task (stable), pad every segment to a multiple of 4 slots
    std::vector<int32_t> seg_len(T, 0), seg_off((size_t)T + 1, 0);
    for (int64_t v = 0; v < V; ++v) seg_len[task_id[v]] += 1;
    int64_t total = 0;
    int32_t max_seg = 0, max_lds_seg = 0, wide = 0;
    for (int32_t t = 0; t < T; ++t) {
        seg_off[t] = (int32_t)total;
        total += (seg_len[t] + 3) & ~3;
        if (total > INT32_MAX - 64) return INFAAS_SEL_ERR_INVALID_ARG;
        max_seg = std::max(max_seg, seg_len[t]);
        if (seg_len[t] > h->lds_limit) wide += 1;
        else max_lds_seg = std::max(max_lds_seg, seg_len[t]);
    }
    seg_off[T] = (int32_t)total;
    const int32_t Vp = (int32_t)((total + 63) & ~(int64_t)63) + 64;

    std::vector<int32_t> acc(Vp, INT32_MIN), queue(Vp, INT32_MAX), orig(Vp, -1), slot_of(std::max(V, 1), 0);
    std::vector<int32_t> lat((size_t)B * Vp, INT32_MAX);
    std::vector<uint32_t> rank((size_t)B * Vp, kNoRank), perm((size_t)B * Vp, 0u);
    std::vector<int32_t> acc_r((size_t)B * Vp, INT32_MIN), orig_r((size_t)B * Vp, -1);
    std::vector<uint32_t> tot_r((size_t)B * Vp, 0xFFFFFFFFu);
    {
        std::vector<int32_t> fill(T, 0);
        for (int64_t v = 0; v < V; ++v) {
            int32_t t = task_id[v];
            int32_t slot = seg_off[t] + fill[t]++;
            acc[slot] = acc_bp[v];
            queue[slot] = queue_us[v];
            orig[slot] = (int32_t)v;
            slot_of[v] = slot;
            for (int32_t b = 0; b < B; ++b) lat[(size_t)b * Vp + slot] = lat_us[v * B + b];
        }
    }
    // ---- rank of every row inside its (task, batch) slice under (cost, latency, row)
    {
        std::vector<int32_t> ord;
        for (int32_t t = 0; t < T; ++t) {
            const int32_t L = seg_len[t], seg = seg_off[t];
            if (L == 0) continue;
            ord.resize(L);
            for (int32_t b = 0; b < B; ++b) {
                std::iota(ord.begin(), ord.end(), 0);
                std::sort(ord.begin(), ord.end(), [&](int32_t x, int32_t y) {
                    const int64_t vx = orig[seg + x], vy = orig[seg + y];
                    const int32_t cx = cost[vx * B + b], cy = cost[vy * B + b];
                    if (cx != cy) return cx < cy;
                    const int32_t lx = lat_us[vx * B + b], ly = lat_us[vy * B + b];
                    if (lx != ly) return lx < ly;
                    return vx < vy;
                });
                for (int32_t r = 0; r < L; ++r) {
                    const size_t g = (size_t)b * Vp + seg + r, sl = (size_t)b * Vp + seg + ord[r];
                    perm[g] = (uint32_t)ord[r];
                    rank[sl] = (uint32_t)r;
                    acc_r[g] = acc[seg + ord[r]];
                    tot_r[g] = (uint32_t)lat[sl] + (uint32_t)queue[seg + ord[r]];
                    orig_r[g] = orig[seg + ord[r]];
                }
            }
        }
    }

    // ---- upload
    DeviceGuard g(h->device);
    if (!g.ok) return INFAAS_SEL_ERR_HIP;
    if (!HIP_OK(hipDeviceSynchronize())) return INFAAS_SEL_ERR_HIP;
    h->free_table();
    bool ok = dev_alloc(&h->d_acc, Vp) == hipSuccess && dev_alloc(&h->d_queue, Vp) == hipSuccess &&
              dev_alloc(&h->d_orig, Vp) == hipSuccess && dev_alloc(&h->d_lat, (size_t)B * Vp) == hipSuccess &&
              dev_alloc(&h->d_rank, (size_t)B * Vp) == hipSuccess &&
              dev_alloc(&h->d_perm, (size_t)B * Vp) == hipSuccess &&
              dev_alloc(&h->d_seg_off, (size_t)T + 1) == hipSuccess && dev_alloc(&h->d_seg_len, T) == hipSuccess &&
              dev_alloc(&h->d_slot_of, std::max(V, 1)) == hipSuccess &&
              dev_alloc(&h->d_acc_r, (size_t)B * Vp) == hipSuccess && dev_alloc(&h->d_orig_r, (size_t)B * Vp) == hipSuccess &&
              dev_alloc(&h->d_row_entry, (size_t)std::max(V, 1) * B) == hipSuccess &&
              dev_alloc(&h->d_tot_r, (size_t)B * Vp) == hipSuccess;
    if (!ok) {
        h->free_table();
        (void)hipGetLastError();
        return INFAAS_SEL_ERR_OOM;
    }
    auto up = [](void *d, const void *s, size_t bytes) {
        return bytes == 0 || HIP_OK(hipMemcpy(d, s, bytes, hipMemcpyHostToDevice));
    };
    ok = up(h->d_acc, acc.data(), (size_t)Vp * 4) && up(h->d_queue, queue.data(), (size_t)Vp * 4) &&
         up(h->d_orig, orig.data(), (size_t)Vp * 4) && up(h->d_lat, lat.data(), (size_t)B * Vp * 4) &&
         up(h->d_rank, rank.data(), (size_t)B * Vp * 4) && up(h->d_perm, perm.data(), (size_t)B * Vp * 4) &&
         up(h->d_seg_off, seg_off.data(), ((size_t)T + 1) * 4) && up(h->d_seg_len, seg_len.data(), (size_t)T * 4) &&
         up(h->d_slot_of, slot_of.data(), (size_t)std::max(V, 1) * 4) &&
         up(h->d_acc_r, acc_r.data(), (size_t)B * Vp * 4) && up(h->d_orig_r, orig_r.data(), (size_t)B * Vp * 4) &&
         up(h->d_tot_r, tot_r.data(), (size_t)B * Vp * 4);
    if (!ok) {
        h->free_table();
        return INFAAS_SEL_ERR_HIP;
    }
    h->V = V;
    h->Vp = Vp;
    h->max_segment = max_seg;
    h->max_lds_segment = max_lds_seg;
    h->wide_segments = wide;
    h->table_bytes = (int64_t)Vp * 4 * (3 + 6 * (int64_t)B) + (int64_t)std::max(V, 1) * B * 8 + ((int64_t)2 * T + 1 + std::max(V, 1)) * 4;
    TableView tv{};
    tv.T = T; tv.B = B; tv.S = T * B; tv.V = V; tv.Vp = Vp; tv.lds_limit = h->lds_limit; tv.max_len = max_seg;
    tv.acc = h->d_acc; tv.queue = h->d_queue; tv.orig = h->d_orig; tv.lat = h->d_lat;
    tv.rank = h->d_rank; tv.perm = h->d_perm; tv.seg_off = h->d_seg_off; tv.seg_len = h->d_seg_len;
    tv.slot_of = h->d_slot_of;
    tv.acc_r = h->d_acc_r; tv.tot_r = h->d_tot_r; tv.orig_r = h->d_orig_r;
    tv.row_entry = h->d_row_entry;
    tv.acc_base = 0;
    for (int64_t v = 0; v < V; ++v) tv.acc_base = (v == 0 || acc_bp[v] < tv.acc_base) ? acc_bp[v] : tv.acc_base;
    // the lookup forms acc_base - 1; a slice that holds the one accuracy below this base is not indexed
    if (tv.acc_base == INT32_MIN) tv.acc_base = INT32_MIN + 1;
    tv.state = nullptr;
    tv.want_state = 1;
    if (!HIP_OK(launch_row_entries(tv, nullptr))) {
        h->free_table();
        return INFAAS_SEL_ERR_HIP;
    }
    h->tv = tv;
    h->h_task.swap(keep_task); h->h_acc.swap(keep_acc); h->h_lat.swap(keep_lat);
    h->loaded = true;
    if ((h->flags & INFAAS_SEL_ENGINE_MASK) != INFAAS_SEL_ENGINE_SCAN) {
        int rc = create_index(h);
        if (rc != INFAAS_SEL_OK) {
            h->free_table();
            return rc;
        }
    }
    if (!h->have_index && !HIP_OK(hipDeviceSynchronize())) {   // (the index build has waited for row_entry)
        h->free_table();
        return INFAAS_SEL_ERR_HIP;
    }
    return INFAAS_SEL_OK;
}

namespace {

// Whether what is enqueued on st is recorded into a graph instead of run (also where the runtime cannot tell).  id: number of
// the capture, 0 without one and where it is not known.
bool is_captured(hipStream_t st, unsigned long long *id = nullptr)
{
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    const bool known = (id ? hipStreamGetCaptureInfo(st, &capture, id) : hipStreamIsCapturing(st, &capture)) == hipSuccess;
    if (!known) (void)hipGetLastError();
    if (id && (!known || capture == hipStreamCaptureStatusNone)) *id = 0;
    return !known || capture != hipStreamCaptureStatusNone;
}
// To be called for every report; whether it is only recorded.  A recorded one arrives with every replay of its graph, behind the
// back of the marks above: as long as the same capture records no refresh behind it, nothing counts as up to date.
bool note_report(infaas_sel *h, hipStream_t st)
{
    h->refreshed_in = 0;
    unsigned long long id = 0;
    if (!is_captured(st, &id)) return false;
    h->replays = h->replays || id == 0 || (h->reported_in != 0 && h->reported_in != id);
    h->reported_in = id;
    return true;
}
bool may_be_replayed(const infaas_sel *h) { return h->replays || h->reported_in != 0; }

}  // namespace

int infaas_sel_update_load(infaas_sel_t *h, int32_t n, const int32_t *d_variant_idx,
                           const int32_t *d_queue_us, void *hip_stream)
{
    if (!h || n < 0) return INFAAS_SEL_ERR_INVALID_ARG;
    if (!h->loaded) return INFAAS_SEL_ERR_NOT_LOADED;
    if (n == 0) return INFAAS_SEL_OK;
    if (!d_variant_idx || !d_queue_us) return INFAAS_SEL_ERR_INVALID_ARG;
    DeviceGuard g(h->device);
    if (!g.ok) return INFAAS_SEL_ERR_HIP;
    hipStream_t st = (hipStream_t)hip_stream;
    {
        LaunchTimer t(h, INFAAS_SEL_K_UPDATE, st);
        if (!HIP_OK(launch_update_load(h->tv, n, d_variant_idx, d_queue_us,
                                       h->have_index ? &h->ix : nullptr, st, t.ev())))
            return INFAAS_SEL_ERR_HIP;
    }
    if (h->have_index) {  // the steps depend on the load: rebuild them behind the update
        h->steps_stale = true;
        note_report(h, st);
        LaunchTimer t(h, INFAAS_SEL_K_INDEX_BUILD, st);
        if (!HIP_OK(launch_index_build(h->tv, h->ix, st, t.ev()))) return INFAAS_SEL_ERR_HIP;
    }
    return INFAAS_SEL_OK;
}

namespace {

// A state report (idx null: of all rows) on the tables of both tiers, whose indexes are rebuilt behind it.
// derive: the states are those the instances' states give.
int apply_states(infaas_sel *h, infaas_sel *sub, bool derive, int32_t n, const int32_t *d_idx, const int32_t *d_states, hipStream_t st)
{
    {
        LaunchTimer t(h, INFAAS_SEL_K_UPDATE_STATE, st);
        const hipError_t e = derive ? launch_derive_states(h->wv, h->tv, h->ix, sub->tv, sub->ix, st, t.ev())
                                    : launch_update_state(h->tv, h->ix, sub->tv, sub->ix, n, d_idx, d_states, st, t.ev());
        if (!HIP_OK(e)) return INFAAS_SEL_ERR_HIP;
    }
    h->steps_stale = sub->steps_stale = true;
    const bool captured = note_report(h, st);
    if (derive) {   // it has gone through loads and utilisations, too
        h->workers_dirty = captured;
        h->rows_stale = true;
    }
    IndexView ia = h->ix, ib = sub->ix;
    // The build leaves the steps' workers behind when the worker of every variant is up to date.  (Not in a graph: what is
    // captured has not happened yet, and a call in front of the first replay must not rely on it.)
    const bool fill = h->workers_loaded && !h->workers_dirty && !captured && !may_be_replayed(h);
    if (fill) {
        ia.fill.by_row = h->wv.row_worker;
        ib.fill.cls = h->wv.var_cls; ib.fill.best = h->wv.best_cls;
        if (h->rows_stale) ib.fill.rows = h->wv.row_worker + h->V;
    }
    LaunchTimer t(h, INFAAS_SEL_K_INDEX_BUILD, st);
    if (!HIP_OK(launch_index_build(h->tv, ia, sub->tv, ib, st, t.ev()))) return INFAAS_SEL_ERR_HIP;
    if (fill) h->steps_stale = sub->steps_stale = h->rows_stale = false;
    return INFAAS_SEL_OK;
}

}  // namespace

int infaas_sel_load_states(infaas_sel_t *h, const int32_t *state, const int32_t *load_us)
{
    if (!h) return INFAAS_SEL_ERR_INVALID_ARG;
    if (!h->loaded) return INFAAS_SEL_ERR_NOT_LOADED;
    if (!h->have_index || (h->V > 0 && (!state || !load_us))) return INFAAS_SEL_ERR_INVALID_ARG;
    const int32_t V = h->V, B = h->B;
    std::vector<int32_t> combined((size_t)V * B);   // load + inference latency: the Inactive tier's order
    for (int64_t v = 0; v < V; ++v) {
        if (state[v] < 0 || state[v] > 3 || load_us[v] < 0) return INFAAS_SEL_ERR_OUT_OF_RANGE;
        for (int32_t b = 0; b < B; ++b) {
            const int64_t c = (int64_t)load_us[v] + h->h_lat[(size_t)v * B + b];
            if (c > INT32_MAX) return INFAAS_SEL_ERR_OUT_OF_RANGE;
            combined[(size_t)v * B + b] = (int32_t)c;
        }
    }
    DeviceGuard g(h->device);
    if (!g.ok) return INFAAS_SEL_ERR_HIP;
    if (!HIP_OK(hipDeviceSynchronize())) return INFAAS_SEL_ERR_HIP;
    h->drop_inactive();
    // The Inactive tier is a table of its own over the same rows: cost := load + latency (its order
    // is (load + latency, latency, row)) and queue := load (its latency test is load + latency <= slo).
    infaas_sel_config cfg{};
    cfg.num_tasks = h->T; cfg.num_batch_sizes = B; cfg.batch_sizes = h->batch_sizes.data();
    cfg.device = h->device; cfg.flags = INFAAS_SEL_ENGINE_INDEX; cfg.lds_segment_limit = h->lds_limit;
    infaas_sel *sub = nullptr;
    int rc = infaas_sel_create(&cfg, &sub);
    if (rc == INFAAS_SEL_OK)
        rc = infaas_sel_load_variants(sub, V, h->h_task.data(), h->h_acc.data(), h->h_lat.data(), combined.data(), load_us);
    if (rc == INFAAS_SEL_OK && !sub->have_index) rc = INFAAS_SEL_ERR_INVALID_ARG;
    int32_t *d_states = nullptr;
    if (rc == INFAAS_SEL_OK) {
        const size_t rows = (size_t)std::max(V, 1);
        if (!h->d_state && dev_alloc(&h->d_state, rows) != hipSuccess) rc = INFAAS_SEL_ERR_OOM;
        if (rc == INFAAS_SEL_OK && dev_alloc(&sub->d_state, rows) != hipSuccess) rc = INFAAS_SEL_ERR_OOM;
        if (rc == INFAAS_SEL_OK && dev_alloc(&d_states, rows) != hipSuccess) rc = INFAAS_SEL_ERR_OOM;
        if (rc == INFAAS_SEL_ERR_OOM) (void)hipGetLastError();
    }
    if (rc == INFAAS_SEL_OK) {
        // a state that is none, so that every row's is seen to change
        if (!HIP_OK(hipMemset(h->d_state, 0x7F, (size_t)V * 4)) || !HIP_OK(hipMemset(sub->d_state, 0x7F, (size_t)V * 4)) ||
            (V > 0 && !HIP_OK(hipMemcpy(d_states, state, (size_t)V * 4, hipMemcpyHostToDevice))))
            rc = INFAAS_SEL_ERR_HIP;
    }
    if (rc == INFAAS_SEL_OK) {
        h->tv.state = h->d_state; h->tv.want_state = 1;       // Active
        sub->tv.state = sub->d_state; sub->tv.want_state = 0; // Inactive
        rc = apply_states(h, sub, false, V, nullptr, d_states, nullptr);
        if (rc == INFAAS_SEL_OK && !HIP_OK(hipDeviceSynchronize())) rc = INFAAS_SEL_ERR_HIP;
    }
    (void)hipFree(d_states);
    if (rc != INFAAS_SEL_OK) {
        if (sub) infaas_sel_destroy(sub);
        // the states may have been applied to this table's columns already: rather than leave a
        // table that silently answers from some of its variants, drop it
        (void)hipDeviceSynchronize();
        h->free_table();
        return rc;
    }
    sub->timing = h->timing;
    h->inactive = sub;
    return INFAAS_SEL_OK;
}

int infaas_sel_update_state(infaas_sel_t *h, int32_t n, const int32_t *d_variant_idx,
                            const int32_t *d_state, void *hip_stream)
{
    if (!h || n < 0) return INFAAS_SEL_ERR_INVALID_ARG;
    if (!h->loaded || !h->inactive) return INFAAS_SEL_ERR_NOT_LOADED;
    if (h->instance_states) return INFAAS_SEL_ERR_INVALID_ARG;   // a variant's state follows from its instances now
    if (n == 0) return INFAAS_SEL_OK;
    if (!d_variant_idx || !d_state) return INFAAS_SEL_ERR_INVALID_ARG;
    DeviceGuard g(h->device);
    if (!g.ok) return INFAAS_SEL_ERR_HIP;
    return apply_states(h, h->inactive, false, n, d_variant_idx, d_state, (hipStream_t)hip_stream);
}

namespace {

// Common part of the two select calls; d_out_closest is null for the plain one.
int select_impl(infaas_sel_t *h, int64_t N, const int32_t *d_task, const int32_t *d_slo_us,
                const int32_t *d_min_acc_bp, const int32_t *d_batch_idx, int32_t *d_out_variant,
                int32_t *d_out_closest, bool closest, void *hip_stream)
{
    if (!h || N < 0) return INFAAS_SEL_ERR_INVALID_ARG;
    if (!h->loaded) return INFAAS_SEL_ERR_NOT_LOADED;
    if (closest && h->inactive) {
        snprintf(g_last_error, sizeof(g_last_error),
                 "infaas_sel_select_closest needs a handle without variant states (with states: infaas_sel_select_tiered_closest)");
        return INFAAS_SEL_ERR_INVALID_ARG;
    }
    if (N == 0) return INFAAS_SEL_OK;
    if (!d_task || !d_slo_us || !d_min_acc_bp || !d_batch_idx || !d_out_variant || (closest && !d_out_closest))
        return INFAAS_SEL_ERR_INVALID_ARG;
    DeviceGuard g(h->device);
    if (!g.ok) return INFAAS_SEL_ERR_HIP;
    hipStream_t st = (hipStream_t)hip_stream;
    // (with variant states only the index honours them: its columns are masked, the scan's are not)
    // (the suggestion comes from the index whenever there is one; without one, from an exhaustive scan behind
    // the scan engine's selection)
    const bool idx = (closest && h->have_index) || h->inactive != nullptr || use_index(h);
    const bool ranked = !idx && use_ranked(h);
    int rc = idx || ranked ? INFAAS_SEL_OK : ensure_scratch(h, std::min(N, kMaxPass));
    if (rc != INFAAS_SEL_OK) return rc;
    for (int64_t done = 0; done < N; done += kMaxPass) {
        QueryView q{};
        q.n = (int32_t)std::min(kMaxPass, N - done);
        q.task = d_task + done; q.slo = d_slo_us + done; q.min_acc = d_min_acc_bp + done;
        q.bidx = d_batch_idx + done; q.out = d_out_variant + done;
        q.closest = closest ? d_out_closest + done : nullptr;
        q.pass = closest ? 1 : 0;
        rc = idx ? index_pass(h, q, st) : ranked ? ranked_pass(h, q, st) : scan_pass(h, q, st);
        if (rc != INFAAS_SEL_OK) return rc;
        if (closest && !idx) {
            LaunchTimer t(h, INFAAS_SEL_K_CLOSEST_SCAN, st);
            if (!HIP_OK(launch_closest_scan(h->tv, q, h->num_cus, st, t.ev()))) return INFAAS_SEL_ERR_HIP;
        }
    }
    h->last_stats = idx ? h->ix.stats : nullptr;
    return INFAAS_SEL_OK;
}

}  // namespace

int infaas_sel_select(infaas_sel_t *h, int64_t N, const int32_t *d_task, const int32_t *d_slo_us,
                      const int32_t *d_min_acc_bp, const int32_t *d_batch_idx,
                      int32_t *d_out_variant, void *hip_stream)
{
    return select_impl(h, N, d_task, d_slo_us, d_min_acc_bp, d_batch_idx, d_out_variant, nullptr, false, hip_stream);
}

namespace {

// Brings the worker of every variant, then of every step of both indexes, up to date.  What is only recorded into a graph
// has not happened yet: it serves the calls recorded behind it, and an eager one does it again.
int refresh_workers(infaas_sel *h, hipStream_t st)
{
    infaas_sel *sub = h->inactive;
    if (!h->workers_dirty && !h->rows_stale && !h->steps_stale && !sub->steps_stale && !may_be_replayed(h)) return INFAAS_SEL_OK;
    unsigned long long id = 0;
    const bool captured = is_captured(st, &id);
    if (captured && id != 0 && id == h->refreshed_in) return INFAAS_SEL_OK;
    // (of the reports that this capture has recorded itself the marks tell)
    const bool unknown = h->replays || (h->reported_in != 0 && h->reported_in != id);
    const bool tables = unknown || h->workers_dirty, rows = tables || h->rows_stale, a = tables || h->steps_stale, b = tables || sub->steps_stale;
    if (tables) {
        LaunchTimer t(h, INFAAS_SEL_K_WORKER_TABLES, st);
        if (!HIP_OK(launch_worker_tables(h->wv, st, t.ev()))) return INFAAS_SEL_ERR_HIP;
    }
    {
        LaunchTimer t(h, INFAAS_SEL_K_STEP_WORKERS, st);
        if (!HIP_OK(launch_step_workers(h->wv, a ? &h->ix : nullptr, b ? &sub->ix : nullptr, h->T * h->B, rows, st, t.ev())))
            return INFAAS_SEL_ERR_HIP;
    }
    if (captured) {
        h->refreshed_in = id;
        if (h->reported_in == id) h->reported_in = 0;
        return INFAAS_SEL_OK;
    }
    h->workers_dirty = h->rows_stale = h->steps_stale = sub->steps_stale = false;
    return INFAAS_SEL_OK;
}

// The state-aware selection, with the worker of every answer when d_out_worker is given and with
// the closest variant for the queries neither tier answers when d_out_closest is given.
int tiered_impl(infaas_sel_t *h, int64_t N, const int32_t *d_task, const int32_t *d_slo_us,
                const int32_t *d_min_acc_bp, const int32_t *d_batch_idx,
                int32_t *d_out_variant, int32_t *d_out_tier, int32_t *d_out_worker, bool workers, void *hip_stream,
                int32_t *d_out_closest = nullptr, bool closest = false)
{
    if (!h || N < 0) return INFAAS_SEL_ERR_INVALID_ARG;
    if (!h->loaded || !h->inactive || (workers && !h->workers_loaded)) return INFAAS_SEL_ERR_NOT_LOADED;
    if (N == 0) return INFAAS_SEL_OK;
    if (!d_task || !d_slo_us || !d_min_acc_bp || !d_batch_idx || !d_out_variant || !d_out_tier ||
        (workers && !d_out_worker) || (closest && !d_out_closest))
        return INFAAS_SEL_ERR_INVALID_ARG;
    DeviceGuard g(h->device);
    if (!g.ok) return INFAAS_SEL_ERR_HIP;
    hipStream_t st = (hipStream_t)hip_stream;
    // One kernel against two mirrors and two launches.
    const IndexShape xa = shape_of(h), xb = shape_of(h->inactive);
    bool direct = memory_pays(xa, &xb, workers, closest, N);
    // The lists are allocated for direct calls too: the choice follows the index, and the same call after a report
    // may need them where nothing can be allocated (under capture, after an eager call to warm up).  A call that is
    // itself captured and finds none does without.
    const int64_t most = std::min(N, kMaxTierPass);
    int rc = INFAAS_SEL_OK;
    if (!open_there(h, most, closest)) {
        if (is_captured(st)) direct = true;
        else rc = ensure_open(h, most, closest);
    }
    if (rc == INFAAS_SEL_OK && workers) rc = refresh_workers(h, st);
    if (rc != INFAAS_SEL_OK) return rc;
    // The Active tier's lookup writes all result arrays and lists the valid queries it could not
    // answer; the Inactive tier's lookup reads only those lists and fills in what it can answer.
    for (int64_t done = 0; done < N; done += kMaxTierPass) {
        QueryView q{};
        q.n = (int32_t)std::min(kMaxTierPass, N - done);
        q.task = d_task + done; q.slo = d_slo_us + done; q.min_acc = d_min_acc_bp + done;
        q.bidx = d_batch_idx + done; q.out = d_out_variant + done; q.tier = d_out_tier + done;
        q.open = h->d_open; q.open_count = h->d_open_count;
        q.open_side = closest ? h->d_open + h->open_words : nullptr;
        q.open_cap = index_open_cap(q.n, h->num_cus);
        if (workers) { q.worker = d_out_worker + done; q.row_worker = h->wv.row_worker; }
        if (closest) q.closest = d_out_closest + done;
        h->last_route = INFAAS_SEL_ROUTE_MEMORY;
        if (direct) {
            LaunchTimer t(h, INFAAS_SEL_K_INDEX_SELECT, st);
            if (!HIP_OK(launch_direct_modes(h->tv, h->ix, h->inactive->tv, h->inactive->ix, q, true, xa.open > 0 || xb.open > 0, h->num_cus, st, t.ev())))
                return INFAAS_SEL_ERR_HIP;
            continue;
        }
        q.pass = workers ? (closest ? 8 : 4) : closest ? 6 : 2;
        rc = index_pass(h, q, st);
        if (rc != INFAAS_SEL_OK) return rc;
        if (workers) q.row_worker = h->wv.row_worker + h->V;
        q.pass = workers ? (closest ? 9 : 5) : closest ? 7 : 3;
        rc = index_pass(h->inactive, q, st);
        if (rc != INFAAS_SEL_OK) return rc;
    }
    h->last_stats = h->inactive->ix.stats;
    return INFAAS_SEL_OK;
}

}  // namespace

int infaas_sel_select_tiered(infaas_sel_t *h, int64_t N, const int32_t *d_task, const int32_t *d_slo_us,
                             const int32_t *d_min_acc_bp, const int32_t *d_batch_idx,
                             int32_t *d_out_variant, int32_t *d_out_tier, void *hip_stream)
{
    return tiered_impl(h, N, d_task, d_slo_us, d_min_acc_bp, d_batch_idx, d_out_variant, d_out_tier, nullptr, false,
                       hip_stream);
}

int infaas_sel_select_tiered_closest(infaas_sel_t *h, int64_t N, const int32_t *d_task, const int32_t *d_slo_us,
                                     const int32_t *d_min_acc_bp, const int32_t *d_batch_idx,
                                     int32_t *d_out_variant, int32_t *d_out_tier, int32_t *d_out_closest, void *hip_stream)
{
    return tiered_impl(h, N, d_task, d_slo_us, d_min_acc_bp, d_batch_idx, d_out_variant, d_out_tier, nullptr, false,
                       hip_stream, d_out_closest, true);
}

int infaas_sel_select_workers(infaas_sel_t *h, int64_t N, const int32_t *d_task, const int32_t *d_slo_us,
                              const int32_t *d_min_acc_bp, const int32_t *d_batch_idx,
                              int32_t *d_out_variant, int32_t *d_out_tier, int32_t *d_out_worker, void *hip_stream)
{
    return tiered_impl(h, N, d_task, d_slo_us, d_min_acc_bp, d_batch_idx, d_out_variant, d_out_tier, d_out_worker, true,
                       hip_stream);
}

int infaas_sel_select_workers_closest(infaas_sel_t *h, int64_t N, const int32_t *d_task, const int32_t *d_slo_us,
                                      const int32_t *d_min_acc_bp, const int32_t *d_batch_idx,
                                      int32_t *d_out_variant, int32_t *d_out_tier, int32_t *d_out_worker,
                                      int32_t *d_out_closest, void *hip_stream)
{
    return tiered_impl(h, N, d_task, d_slo_us, d_min_acc_bp, d_batch_idx, d_out_variant, d_out_tier, d_out_worker, true,
                       hip_stream, d_out_closest, true);
}

int infaas_sel_load_workers(infaas_sel_t *h, int32_t num_workers, const int32_t *worker_hw, const int32_t *worker_util,
                            const int32_t *variant_hw, int32_t num_instances, const int32_t *inst_variant,
                            const int32_t *inst_worker, const int32_t *inst_load)
{
    if (!h || num_workers < 0 || num_instances < 0) return INFAAS_SEL_ERR_INVALID_ARG;
    if (!h->loaded || !h->inactive) return INFAAS_SEL_ERR_NOT_LOADED;
    const int32_t V = h->V, W = num_workers, I = num_instances;
    if ((W > 0 && (!worker_hw || !worker_util)) || (V > 0 && !variant_hw) ||
        (I > 0 && (!inst_variant || !inst_worker || !inst_load)))
        return INFAAS_SEL_ERR_INVALID_ARG;
    for (int32_t w = 0; w < W; ++w)
        if (worker_util[w] < 0) return INFAAS_SEL_ERR_OUT_OF_RANGE;
    for (int32_t i = 0; i < I; ++i)
        if (inst_variant[i] < 0 || inst_variant[i] >= V || inst_worker[i] < 0 || inst_worker[i] >= W || inst_load[i] < 0)
            return INFAAS_SEL_ERR_OUT_OF_RANGE;
    // hardware classes that have workers, numbered in ascending order of the caller's codes
    std::vector<int32_t> codes(worker_hw, worker_hw + W);
    std::sort(codes.begin(), codes.end());
    codes.erase(std::unique(codes.begin(), codes.end()), codes.end());
    const int32_t H = (int32_t)codes.size();
    auto class_of = [&](int32_t code) -> int32_t {
        auto it = std::lower_bound(codes.begin(), codes.end(), code);
        return it != codes.end() && *it == code ? (int32_t)(it - codes.begin()) : -1;
    };
    std::vector<int32_t> cls_off((size_t)H + 1, 0), cls_worker((size_t)W), var_cls((size_t)V);
    for (int32_t w = 0; w < W; ++w) cls_off[(size_t)class_of(worker_hw[w]) + 1] += 1;
    for (int32_t c = 0; c < H; ++c) cls_off[(size_t)c + 1] += cls_off[(size_t)c];
    {
        std::vector<int32_t> at(cls_off.begin(), cls_off.end() - 1);
        for (int32_t w = 0; w < W; ++w) cls_worker[(size_t)at[(size_t)class_of(worker_hw[w])]++] = w;
    }
    for (int32_t v = 0; v < V; ++v) var_cls[(size_t)v] = class_of(variant_hw[v]);
    // instances grouped by variant
    std::vector<int32_t> inst_off((size_t)V + 1, 0), inst_w((size_t)I), inst_l((size_t)I), inst_pos((size_t)I);
    for (int32_t i = 0; i < I; ++i) inst_off[(size_t)inst_variant[i] + 1] += 1;
    for (int32_t v = 0; v < V; ++v) inst_off[(size_t)v + 1] += inst_off[(size_t)v];
    {
        std::vector<int32_t> at(inst_off.begin(), inst_off.end() - 1);
        for (int32_t i = 0; i < I; ++i) {
            const int32_t p = at[(size_t)inst_variant[i]]++;
            inst_w[(size_t)p] = inst_worker[i]; inst_l[(size_t)p] = inst_load[i]; inst_pos[(size_t)i] = p;
        }
    }
    DeviceGuard g(h->device);
    if (!g.ok) return INFAAS_SEL_ERR_HIP;
    if (!HIP_OK(hipDeviceSynchronize())) return INFAAS_SEL_ERR_HIP;
    for (void *p : h->worker_mem) (void)hipFree(p);
    h->worker_mem.clear();
    h->workers_loaded = false;
    h->instance_states = false;
    bool ok = true;
    auto upload = [&](const std::vector<int32_t> &src, size_t count) -> int32_t * {
        int32_t *d = nullptr;
        if (!ok) return nullptr;
        if (dev_alloc(&d, count) != hipSuccess) { ok = false; (void)hipGetLastError(); return nullptr; }
        h->worker_mem.push_back(d);
        if (!src.empty() && !HIP_OK(hipMemcpy(d, src.data(), src.size() * 4, hipMemcpyHostToDevice))) ok = false;
        return d;
    };
    WorkerView wv{};
    wv.V = V; wv.W = W; wv.I = I; wv.H = H;
    wv.util = upload(std::vector<int32_t>(worker_util, worker_util + W), (size_t)W);
    wv.cls_off = upload(cls_off, cls_off.size());
    wv.cls_worker = upload(cls_worker, (size_t)W);
    wv.var_cls = upload(var_cls, (size_t)V);
    wv.inst_off = upload(inst_off, inst_off.size());
    wv.inst_worker = upload(inst_w, (size_t)I);
    wv.inst_load = upload(inst_l, (size_t)I);
    wv.inst_pos = upload(inst_pos, (size_t)I);
    wv.best_cls = upload({}, (size_t)H);
    wv.row_worker = upload({}, (size_t)2 * V);
    for (infaas_sel *t : {h, h->inactive}) {
        if (ok && !t->ix.step_worker && dev_alloc(&t->ix.step_worker, t->ix.step_cap) != hipSuccess) {
            ok = false;
            (void)hipGetLastError();
        }
        // 16-bit copies of the workers of the hot steps, for the lookup kernel's LDS
        (void)hipFree(t->ix.hot_worker);
        t->ix.hot_worker = nullptr;
        const size_t hot = (size_t)t->T * t->B * t->ix.hot_rows;
        if (ok && hot > 0 && t->index_lds_bytes > 0 && W <= 65535 &&
            dev_alloc(&t->ix.hot_worker, hot + 8) != hipSuccess) {
            ok = false;
            (void)hipGetLastError();
        }
        t->steps_stale = true;
    }
    if (!ok) {
        for (void *p : h->worker_mem) (void)hipFree(p);
        h->worker_mem.clear();
        h->wv = WorkerView{};
        return INFAAS_SEL_ERR_OOM;
    }
    h->wv = wv;
    h->workers_loaded = true;
    h->workers_dirty = true;
    h->refreshed_in = 0;
    return INFAAS_SEL_OK;
}

int infaas_sel_update_workers(infaas_sel_t *h, int32_t n, const int32_t *d_worker_idx, const int32_t *d_worker_util,
                              int32_t m, const int32_t *d_inst_idx, const int32_t *d_inst_load, void *hip_stream)
{
    if (!h || n < 0 || m < 0) return INFAAS_SEL_ERR_INVALID_ARG;
    if (!h->loaded || !h->workers_loaded) return INFAAS_SEL_ERR_NOT_LOADED;
    if ((n > 0 && (!d_worker_idx || !d_worker_util)) || (m > 0 && (!d_inst_idx || !d_inst_load)))
        return INFAAS_SEL_ERR_INVALID_ARG;
    if (n == 0 && m == 0) return INFAAS_SEL_OK;
    DeviceGuard g(h->device);
    if (!g.ok) return INFAAS_SEL_ERR_HIP;
    hipStream_t st = (hipStream_t)hip_stream;
    LaunchTimer t(h, INFAAS_SEL_K_WORKER_REPORT, st);
    if (!HIP_OK(launch_worker_report(h->wv, n, d_worker_idx, d_worker_util, m, d_inst_idx, d_inst_load, st, t.ev())))
        return INFAAS_SEL_ERR_HIP;
    h->workers_dirty = true;
    note_report(h, st);
    return INFAAS_SEL_OK;
}

// The variants' states derived anew from the instances', applied to both tiers' tables, both indexes
// rebuilt behind it (as after a state report).
static int apply_instance_states(infaas_sel *h, hipStream_t st) { return apply_states(h, h->inactive, true, 0, nullptr, nullptr, st); }

int infaas_sel_load_instance_states(infaas_sel_t *h, const int32_t *inst_state)
{
    if (!h) return INFAAS_SEL_ERR_INVALID_ARG;
    if (!h->loaded || !h->inactive || !h->workers_loaded) return INFAAS_SEL_ERR_NOT_LOADED;
    const int32_t I = h->wv.I;
    if (I > 0 && !inst_state) return INFAAS_SEL_ERR_INVALID_ARG;
    for (int32_t i = 0; i < I; ++i)
        if (inst_state[i] < INFAAS_SEL_STATE_ACTIVE || inst_state[i] > INFAAS_SEL_STATE_INTERFERED) return INFAAS_SEL_ERR_OUT_OF_RANGE;
    DeviceGuard g(h->device);
    if (!g.ok) return INFAAS_SEL_ERR_HIP;
    if (!HIP_OK(hipDeviceSynchronize())) return INFAAS_SEL_ERR_HIP;
    // in the order the instances are kept in: grouped by variant
    std::vector<int32_t> pos((size_t)I), grouped((size_t)I);
    if (I > 0 && !HIP_OK(hipMemcpy(pos.data(), h->wv.inst_pos, (size_t)I * 4, hipMemcpyDeviceToHost))) return INFAAS_SEL_ERR_HIP;
    for (int32_t i = 0; i < I; ++i) grouped[(size_t)pos[(size_t)i]] = inst_state[i];
    if (!h->wv.inst_state) {
        int32_t *d_st = nullptr;
        if (dev_alloc(&d_st, (size_t)std::max(I, 1)) != hipSuccess) {
            (void)hipGetLastError();
            return INFAAS_SEL_ERR_OOM;
        }
        h->worker_mem.push_back(d_st);
        h->wv.inst_state = d_st;
    }
    if (I > 0 && !HIP_OK(hipMemcpy(h->wv.inst_state, grouped.data(), (size_t)I * 4, hipMemcpyHostToDevice))) return INFAAS_SEL_ERR_HIP;
    h->instance_states = true;
    int rc = apply_instance_states(h, nullptr);
    if (rc == INFAAS_SEL_OK && !HIP_OK(hipDeviceSynchronize())) rc = INFAAS_SEL_ERR_HIP;
    return rc;
}

int infaas_sel_update_instance_states(infaas_sel_t *h, int32_t n, const int32_t *d_inst_idx, const int32_t *d_state,
                                      void *hip_stream)
{
    if (!h || n < 0) return INFAAS_SEL_ERR_INVALID_ARG;
    if (!h->loaded || !h->inactive || !h->workers_loaded || !h->instance_states) return INFAAS_SEL_ERR_NOT_LOADED;
    if (n == 0) return INFAAS_SEL_OK;
    if (!d_inst_idx || !d_state) return INFAAS_SEL_ERR_INVALID_ARG;
    DeviceGuard g(h->device);
    if (!g.ok) return INFAAS_SEL_ERR_HIP;
    hipStream_t st = (hipStream_t)hip_stream;
    {
        LaunchTimer t(h, INFAAS_SEL_K_INSTANCE_STATES, st);
        if (!HIP_OK(launch_instance_state_report(h->wv, n, d_inst_idx, d_state, st, t.ev()))) return INFAAS_SEL_ERR_HIP;
    }
    return apply_instance_states(h, st);
}

int infaas_sel_select_noalloc(infaas_sel_t *h, int64_t N, const int32_t *d_task, const int32_t *d_slo_us,
                              const int32_t *d_min_acc_bp, const int32_t *d_batch_idx,
                              int32_t *d_out_variant, void *hip_stream)
{
    if (!h || N < 0) return INFAAS_SEL_ERR_INVALID_ARG;
    if (!h->loaded) return INFAAS_SEL_ERR_NOT_LOADED;
    if (N > INFAAS_SEL_NOALLOC_MAX_QUERIES) {
        snprintf(g_last_error, sizeof(g_last_error), "infaas_sel_select_noalloc: %lld queries exceed the limit of %lld per call",
                 (long long)N, (long long)INFAAS_SEL_NOALLOC_MAX_QUERIES);
        return INFAAS_SEL_ERR_INVALID_ARG;
    }
    if (!h->have_index || !use_index(h)) {
        snprintf(g_last_error, sizeof(g_last_error),
                 "infaas_sel_select_noalloc needs the staircase index, in automatic mode complete for half of the slices or more");
        return INFAAS_SEL_ERR_INVALID_ARG;
    }
    if (index_park_bytes(h->num_cus) > kStaticScratchBytes) {
        snprintf(g_last_error, sizeof(g_last_error),
                 "infaas_sel_select_noalloc: the static scratch array is sized for %d compute units, this device has %d",
                 kStaticMaxCus, h->num_cus);
        return INFAAS_SEL_ERR_INVALID_ARG;
    }
    if (!h->static_park) {
        snprintf(g_last_error, sizeof(g_last_error), "infaas_sel_select_noalloc: the address of the static scratch array is not known");
        return INFAAS_SEL_ERR_HIP;
    }
    if (N == 0) return INFAAS_SEL_OK;
    if (!d_task || !d_slo_us || !d_min_acc_bp || !d_batch_idx || !d_out_variant) return INFAAS_SEL_ERR_INVALID_ARG;
    DeviceGuard g(h->device);
    if (!g.ok) return INFAAS_SEL_ERR_HIP;
    QueryView q{};
    q.n = (int32_t)N;
    q.task = d_task; q.slo = d_slo_us; q.min_acc = d_min_acc_bp; q.bidx = d_batch_idx; q.out = d_out_variant;
    q.pass = 0;
    // no event pair even when timing is on: taking one may create it
    if (!HIP_OK(launch_select(h, q, h->static_park, (hipStream_t)hip_stream))) return INFAAS_SEL_ERR_HIP;
    h->last_stats = h->ix.stats;
    return INFAAS_SEL_OK;
}

int infaas_sel_select_closest(infaas_sel_t *h, int64_t N, const int32_t *d_task, const int32_t *d_slo_us,
                              const int32_t *d_min_acc_bp, const int32_t *d_batch_idx,
                              int32_t *d_out_variant, int32_t *d_out_closest, void *hip_stream)
{
    return select_impl(h, N, d_task, d_slo_us, d_min_acc_bp, d_batch_idx, d_out_variant, d_out_closest, true,
                       hip_stream);
}

int infaas_sel_load_scaling(infaas_sel_t *h, const int32_t *arch_id, const int32_t *sat_qps, const int32_t *hw_cost,
                            const int32_t *load_us, int32_t lambda_per_s, int32_t slack_pct)
{
    if (!h) return INFAAS_SEL_ERR_INVALID_ARG;
    if (!h->loaded) return INFAAS_SEL_ERR_NOT_LOADED;
    const int32_t V = h->V, B = h->B;
    if (V > 0 && (!arch_id || !sat_qps || !hw_cost || !load_us)) return INFAAS_SEL_ERR_INVALID_ARG;
    if (lambda_per_s < 0 || lambda_per_s > 1000 || slack_pct < 0 || slack_pct > 200) return INFAAS_SEL_ERR_OUT_OF_RANGE;
    for (int32_t v = 0; v < V; ++v)
        if (sat_qps[v] < 1 || hw_cost[v] < 0 || hw_cost[v] > 1048576 || load_us[v] < 0) return INFAAS_SEL_ERR_OUT_OF_RANGE;
    // architectures numbered in ascending order of the caller's codes; their variants, rows ascending
    std::vector<int32_t> by_arch((size_t)V);
    std::iota(by_arch.begin(), by_arch.end(), 0);
    std::stable_sort(by_arch.begin(), by_arch.end(), [&](int32_t a, int32_t b) { return arch_id[a] < arch_id[b]; });
    std::vector<int32_t> arch_first;   // [A + 1] into by_arch
    for (int32_t p = 0; p < V; ++p)
        if (p == 0 || arch_id[by_arch[(size_t)p]] != arch_id[by_arch[(size_t)p - 1]]) arch_first.push_back(p);
    const int32_t A = (int32_t)arch_first.size();
    arch_first.push_back(V);
    auto unit_of = [&](int32_t v) {   // cost of one loaded instance, < 2^62
        return (uint64_t)hw_cost[v] * (1000000ull + (uint64_t)lambda_per_s * (uint64_t)load_us[v]);
    };
    // Candidates of an architecture at a batch size, for scaling up: by descending throughput, and only
    // those that no other variant beats for every request (at least the throughput, at most the latency,
    // and a lower cost per instance or the same with a lower row).  Sorted so that whatever beats a
    // variant comes before it; being beaten is transitive, so the survivors so far are enough to
    // compare with.  Every row of the architecture then gets its block: its own figures and the
    // first candidates of the prefix of the list whose throughput is above its own.
    // For scaling down: by ascending hardware cost, "beats" asks for at most the hardware cost besides
    // (a candidate must be cheaper than the running variant to be one at all), and a row's
    // candidates are the prefix of the list whose hardware cost is below its own.
    if ((int64_t)B * V * kScaleBlockWords * 4 > ((int64_t)1 << 33)) return INFAAS_SEL_ERR_OOM;   // 8 GB of blocks
    std::vector<uint32_t> blocks_of[2];
    std::vector<ScaleCand> cand_of[2];
    std::vector<int32_t> order, cand_cost;
    for (int down = 0; down < 2; ++down) {
        std::vector<uint32_t> &blocks = blocks_of[down];
        std::vector<ScaleCand> &cand = cand_of[down];
        blocks.assign((size_t)std::max<int64_t>((int64_t)B * V, 1) * kScaleBlockWords, 0u);
        // the kernel divides by every throughput and drops what it has no use for: places without a candidate, and the block
        // that an invalid request reads when there are no variants, hold a throughput of 1
        for (size_t w = 0; w < blocks.size(); w += kScaleBlockWords)
            for (int j = -1; j < kScaleInBlock; ++j) blocks[w + (j < 0 ? 0 : 8 + 4 * (size_t)j)] = 1u;
        cand_cost.clear();            // hardware cost of cand[k]
        for (int32_t b = 0; b < B; ++b)
            for (int32_t a = 0; a < A; ++a) {
                order.assign(by_arch.begin() + arch_first[(size_t)a], by_arch.begin() + arch_first[(size_t)a + 1]);
                std::sort(order.begin(), order.end(), [&](int32_t x, int32_t y) {
                    if (!down && sat_qps[x] != sat_qps[y]) return sat_qps[x] > sat_qps[y];
                    if (down && hw_cost[x] != hw_cost[y]) return hw_cost[x] < hw_cost[y];
                    const uint64_t ux = unit_of(x), uy = unit_of(y);
                    if (ux != uy) return ux < uy;
                    return x < y;
                });
                const size_t first = cand.size();
                for (int32_t v : order) {
                    const ScaleCand r{(uint32_t)sat_qps[v], h->h_lat[(size_t)v * B + b], unit_of(v), v, {0, 0, 0}};
                    bool beaten = false;
                    for (size_t k = first; k < cand.size() && !beaten; ++k)
                        beaten = cand[k].qps >= r.qps && cand[k].lat <= r.lat &&
                                 (cand[k].unit < r.unit || (cand[k].unit == r.unit && cand[k].row < v));
                    if (!beaten) { cand.push_back(r); cand_cost.push_back(hw_cost[v]); }
                }
                if (cand.size() > 0x7FFFFFFFull) return INFAAS_SEL_ERR_OUT_OF_RANGE;
                const size_t n = cand.size() - first;
                for (int32_t v : order) {
                    uint32_t *w = &blocks[((size_t)b * V + v) * kScaleBlockWords];
                    const uint64_t unit = unit_of(v);
                    size_t m = 0;   // candidates with a higher throughput, resp. a lower hardware cost: a prefix of the list
                    while (m < n && (down ? cand_cost[first + m] < hw_cost[v] : cand[first + m].qps > (uint32_t)sat_qps[v])) ++m;
                    w[0] = (uint32_t)sat_qps[v]; w[1] = (uint32_t)hw_cost[v];
                    w[2] = (uint32_t)unit; w[3] = (uint32_t)(unit >> 32);
                    w[4] = (uint32_t)h->h_lat[(size_t)v * B + b]; w[5] = (uint32_t)m; w[6] = (uint32_t)first;
                    for (size_t j = 0; j < std::min<size_t>(m, kScaleInBlock); ++j) {
                        const ScaleCand &c = cand[first + j];
                        uint32_t *sl = w + 8 + 4 * j;
                        sl[0] = c.qps; sl[1] = (uint32_t)c.lat; sl[2] = (uint32_t)c.unit; sl[3] = (uint32_t)(c.unit >> 32);
                        w[j < 4 ? 28 + j : 7] = (uint32_t)c.row;
                    }
                }
                // of the list only what no block holds is left
                const auto in_block = (std::ptrdiff_t)std::min<size_t>(n, kScaleInBlock);
                cand.erase(cand.begin() + (std::ptrdiff_t)first, cand.begin() + (std::ptrdiff_t)first + in_block);
                cand_cost.erase(cand_cost.begin() + (std::ptrdiff_t)first, cand_cost.begin() + (std::ptrdiff_t)first + in_block);
            }
        if (cand.empty()) cand.push_back(ScaleCand{1u, 0, 0ull, 0, {0, 0, 0}});
    }
    DeviceGuard g(h->device);
    if (!g.ok) return INFAAS_SEL_ERR_HIP;
    if (!HIP_OK(hipDeviceSynchronize())) return INFAAS_SEL_ERR_HIP;
    for (void *p : h->scale_mem) (void)hipFree(p);
    h->scale_mem.clear();
    h->scaling_loaded = false;
    bool ok = true;
    auto upload = [&](const void *src, size_t bytes) -> void * {
        void *d = nullptr;
        if (!ok) return nullptr;
        if (hipMalloc(&d, std::max<size_t>(bytes, 16)) != hipSuccess) { ok = false; (void)hipGetLastError(); return nullptr; }
        h->scale_mem.push_back(d);
        if (bytes && !HIP_OK(hipMemcpy(d, src, bytes, hipMemcpyHostToDevice))) ok = false;
        return d;
    };
    ScaleView sv{};
    sv.V = V; sv.B = B; sv.slack_pct = slack_pct;
    sv.blocks = (const uint32_t *)upload(blocks_of[0].data(), blocks_of[0].size() * 4);
    sv.cand = (const ScaleCand *)upload(cand_of[0].data(), cand_of[0].size() * sizeof(ScaleCand));
    sv.blocks_down = (const uint32_t *)upload(blocks_of[1].data(), blocks_of[1].size() * 4);
    sv.cand_down = (const ScaleCand *)upload(cand_of[1].data(), cand_of[1].size() * sizeof(ScaleCand));
    if (!ok) {
        for (void *p : h->scale_mem) (void)hipFree(p);
        h->scale_mem.clear();
        return INFAAS_SEL_ERR_OOM;
    }
    h->sv = sv;
    h->scaling_loaded = true;
    return INFAAS_SEL_OK;
}

static int scale_impl(infaas_sel_t *h, bool down, int64_t R, const int32_t *d_variant, const int32_t *d_instances,
                      const int32_t *d_load_qps, const int32_t *d_slo_us, const int32_t *d_batch_idx,
                      int32_t *d_out_action, int32_t *d_out_variant, int32_t *d_out_instances, void *hip_stream)
{
    if (!h || R < 0) return INFAAS_SEL_ERR_INVALID_ARG;
    if (!h->loaded || !h->scaling_loaded) return INFAAS_SEL_ERR_NOT_LOADED;
    if (R == 0) return INFAAS_SEL_OK;
    if (!d_variant || !d_instances || !d_load_qps || !d_slo_us || !d_batch_idx || !d_out_action || !d_out_variant ||
        !d_out_instances)
        return INFAAS_SEL_ERR_INVALID_ARG;
    DeviceGuard g(h->device);
    if (!g.ok) return INFAAS_SEL_ERR_HIP;
    hipStream_t st = (hipStream_t)hip_stream;
    LaunchTimer t(h, down ? INFAAS_SEL_K_SCALE_DOWN : INFAAS_SEL_K_SCALE, st);
    if (!HIP_OK(launch_scale(h->sv, down, R, d_variant, d_instances, d_load_qps, d_slo_us, d_batch_idx, d_out_action,
                             d_out_variant, d_out_instances, h->num_cus, st, t.ev())))
        return INFAAS_SEL_ERR_HIP;
    return INFAAS_SEL_OK;
}

int infaas_sel_scale(infaas_sel_t *h, int64_t R, const int32_t *d_variant, const int32_t *d_instances,
                     const int32_t *d_load_qps, const int32_t *d_slo_us, const int32_t *d_batch_idx,
                     int32_t *d_out_action, int32_t *d_out_variant, int32_t *d_out_instances, void *hip_stream)
{
    return scale_impl(h, false, R, d_variant, d_instances, d_load_qps, d_slo_us, d_batch_idx, d_out_action,
                      d_out_variant, d_out_instances, hip_stream);
}

int infaas_sel_scale_down(infaas_sel_t *h, int64_t R, const int32_t *d_variant, const int32_t *d_instances,
                          const int32_t *d_load_qps, const int32_t *d_slo_us, const int32_t *d_batch_idx,
                          int32_t *d_out_action, int32_t *d_out_variant, int32_t *d_out_instances, void *hip_stream)
{
    return scale_impl(h, true, R, d_variant, d_instances, d_load_qps, d_slo_us, d_batch_idx, d_out_action,
                      d_out_variant, d_out_instances, hip_stream);
}

void infaas_sel_destroy(infaas_sel_t *h)
{
    if (!h) return;
    {
        DeviceGuard g(h->device);
        (void)hipDeviceSynchronize();
        h->free_table();
        h->free_scratch();
        for (auto &p : h->pending) { (void)hipEventDestroy(p.a); (void)hipEventDestroy(p.b); }
        for (auto &e : h->free_events) (void)hipEventDestroy(e);
        if (h->host_stats) (void)hipHostFree(h->host_stats);
    }
    delete h;
}

int infaas_sel_reserve(infaas_sel_t *h, int64_t max_queries)
{
    if (!h || max_queries < 0) return INFAAS_SEL_ERR_INVALID_ARG;
    DeviceGuard g(h->device);
    if (!g.ok) return INFAAS_SEL_ERR_HIP;
    const int64_t cap = std::max<int64_t>(1, std::min(max_queries, kMaxPass));
    if (h->loaded && h->inactive) return ensure_open(h, std::min(cap, kMaxTierPass), h->open_side);
    if (h->loaded && (use_index(h) || use_ranked(h))) return INFAAS_SEL_OK;   // (no scratch per query)
    return ensure_scratch(h, cap);
}

int infaas_sel_read_load(infaas_sel_t *h, int32_t *queue_us, void *hip_stream)
{
    if (!h || !queue_us) return INFAAS_SEL_ERR_INVALID_ARG;
    if (!h->loaded) return INFAAS_SEL_ERR_NOT_LOADED;
    DeviceGuard g(h->device);
    if (!g.ok) return INFAAS_SEL_ERR_HIP;
    if (!HIP_OK(hipStreamSynchronize((hipStream_t)hip_stream))) return INFAAS_SEL_ERR_HIP;
    std::vector<int32_t> q(h->Vp), slot(std::max(h->V, 1));
    if (!HIP_OK(hipMemcpy(q.data(), h->d_queue, (size_t)h->Vp * 4, hipMemcpyDeviceToHost)) ||
        !HIP_OK(hipMemcpy(slot.data(), h->d_slot_of, (size_t)std::max(h->V, 1) * 4, hipMemcpyDeviceToHost)))
        return INFAAS_SEL_ERR_HIP;
    for (int32_t v = 0; v < h->V; ++v) queue_us[v] = q[slot[v]];
    return INFAAS_SEL_OK;
}

int infaas_sel_set_timing(infaas_sel_t *h, int32_t enabled)
{
    if (!h) return INFAAS_SEL_ERR_INVALID_ARG;
    DeviceGuard g(h->device);
    for (auto &p : h->pending) {
        (void)hipEventSynchronize(p.b);
        h->free_events.push_back(p.a);
        h->free_events.push_back(p.b);
    }
    h->pending.clear();
    h->acc = infaas_sel_timings{};
    h->timing = enabled != 0;
    if (h->inactive) return infaas_sel_set_timing(h->inactive, enabled);
    return INFAAS_SEL_OK;
}

int infaas_sel_get_timings(infaas_sel_t *h, infaas_sel_timings *out)
{
    if (!h || !out) return INFAAS_SEL_ERR_INVALID_ARG;
    DeviceGuard g(h->device);
    if (!g.ok) return INFAAS_SEL_ERR_HIP;
    int rc = INFAAS_SEL_OK;
    for (auto &p : h->pending) {
        float ms = 0.f;
        if (hipEventSynchronize(p.b) == hipSuccess && hipEventElapsedTime(&ms, p.a, p.b) == hipSuccess) {
            h->acc.launches[p.kid] += 1;
            h->acc.total_ms[p.kid] += ms;
        } else {   // e.g. the launch itself failed and the events were never attached
            (void)hipGetLastError();
            rc = INFAAS_SEL_ERR_HIP;
        }
        h->free_events.push_back(p.a);
        h->free_events.push_back(p.b);
    }
    h->pending.clear();
    *out = h->acc;
    if (h->inactive) {   // the kernels of the Inactive tier's table count with this handle's
        infaas_sel_timings sub{};
        const int rc2 = infaas_sel_get_timings(h->inactive, &sub);
        for (int k = 0; k < INFAAS_SEL_K_COUNT; ++k) { out->launches[k] += sub.launches[k]; out->total_ms[k] += sub.total_ms[k]; }
        if (rc == INFAAS_SEL_OK) rc = rc2;
    }
    return rc;
}

int infaas_sel_get_info(infaas_sel_t *h, infaas_sel_info *out)
{
    if (!h || !out) return INFAAS_SEL_ERR_INVALID_ARG;
    std::memset(out, 0, sizeof(*out));
    out->num_variants = h->V;
    out->num_slices = h->T * h->B;
    out->max_segment = h->max_segment;
    out->lds_segment_limit = h->lds_limit;
    out->wide_segments = h->wide_segments;
    out->table_bytes = h->table_bytes;
    out->scratch_bytes = h->scratch_bytes + h->park_bytes + h->open_bytes;
    if (h->have_index) {
        out->index_in_lds = h->index_lds_bytes > 0 ? 1 : 0;
        out->index_groups = (int32_t)h->ix.num_groups;
        out->lookup_route = h->last_stats ? h->last_route : 0;
        // (as of the latest build that a selection has run behind, else as loaded)
        const volatile uint32_t *now = h->host_stats;
        out->index_truncated = (int32_t)(now ? now[kCtlTrunc - kCtlMaxK0] + now[kCtlNoBody - kCtlMaxK0]
                                             : h->ix_stats[kCtlTrunc] + h->ix_stats[kCtlNoBody]);
        out->index_max_steps = (int32_t)(now ? now[kCtlMaxK - kCtlMaxK0] : h->ix_stats[kCtlMaxK]);
        out->index_hot_rows = (int32_t)h->ix.hot_rows;
        // (with groups the two counters cover only what lies behind the regions: the figures of the load are kept)
        const bool fresh = now && h->ix.num_groups <= 1;
        const int64_t pool_now = fresh ? (int64_t)now[4] : h->ix_bytes, steps_now = fresh ? (int64_t)now[5] - 1 : h->ix_steps;
        out->index_bytes = pool_now + (int64_t)h->T * h->B * 16 + (steps_now + 1) * 4;
        out->index_steps = steps_now;
        // what the most recent lookup launch did with the queries its first probe could not decide
        std::vector<uint32_t> st((size_t)index_stat_blocks(h->num_cus) * kLookupStats + 1, 0u);   // (its first word: entries in use)
        DeviceGuard g(h->device);
        if (h->last_stats &&
            (!g.ok || !HIP_OK(hipMemcpy(st.data(), h->last_stats - 1, st.size() * 4, hipMemcpyDeviceToHost)))) return INFAAS_SEL_ERR_HIP;
        int64_t sum[kLookupStats] = {0};
        for (size_t i = 0; i < (size_t)st[0] * kLookupStats && i + 1 < st.size(); ++i) sum[i % kLookupStats] += st[i + 1];
        out->lookup_parked = sum[0]; out->lookup_second_body = sum[1]; out->lookup_global_body = sum[2];
        out->lookup_scanned = sum[3]; out->lookup_unanswered = sum[4];
    }
    return INFAAS_SEL_OK;
}

}  // extern "C"
