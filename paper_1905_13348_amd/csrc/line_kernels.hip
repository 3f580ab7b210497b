// The selection (Section 4.1 of the INFaaS paper) for large batches on tables whose staircase index does not fit one compute unit's
// LDS: every query reads the first line of its slice (internal.h), four lanes together, and most have their answer there.
#include "internal.h"
#include "lookup_common.h"

namespace infaas {

namespace {

constexpr int kLineThreads = 1024;
constexpr int kLineQueries = 8;              // per lane and tile
constexpr uint32_t kLineDrain = kLineThreads;                                      // queries set aside that are worth a pass
constexpr uint32_t kLineOpenLds = (kLineDrain + kLineThreads * kLineQueries) * 16;   // a tile may add all of its own

// A workgroup takes a tile of kQueries per lane at a time, and takes it in two phases: first the fields of all of its queries, from HBM, then
// their lines, from L2.  A compute unit's L1 answers in the order in which it was asked, so lines asked for behind fields wait for
// HBM; with the phases of a compute unit apart the two add up only where they must (64M queries on 8000 slices: 440 us with one query per lane
// and as many wavefronts as there are, 640 with the next queries' fields requested while lines are compared, 400 so; with fields that
// are in L2 already 313).  Queries whose first line leaves them open (2% there) are set aside in LDS and finished between two tiles by all
// wavefronts together, when there is one for every lane: the lines that follow, or, for slices with more steps than the index keeps, the search in rank
// order (finished by each wavefront for itself as soon as it had 64, with the others waiting for it at the next tile, 452 us).
// Replaces three passes (binning by groups of tasks whose bodies fit LDS, lookup there, answers back into query order; 48 bytes per query
// instead of 20): 64M queries on 1000 tasks of 100 variants on average 684 us.
__global__ __launch_bounds__(kLineThreads) void k_line_select(TableView tv, IndexView ix, QueryView q, int32_t tile)
{
    extern __shared__ __align__(16) v4i l_open[];   // queries set aside: {query, latency bound, accuracy bound, slice}
    __shared__ uint32_t l_st[kLookupStats], l_count;
    publish_index_stats(tv);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (tid < kLookupStats) l_st[tid] = 0u;
    if (tid == 0) l_count = 0u;
    uint32_t st[kLookupStats] = {0u, 0u, 0u, 0u, 0u};
    const uint32_t row_mask = (1u << ix.line_shift()) - 1u;
    const int32_t acc_base_m1 = tv.acc_base - 1;
    const bool aligned = ((((uintptr_t)q.task) | ((uintptr_t)q.slo) | ((uintptr_t)q.min_acc) | ((uintptr_t)q.bidx) | ((uintptr_t)q.out)) & 15u) == 0;
    constexpr int kGroups = kLineQueries / 4;   // a lane's queries: four consecutive ones in each
    // (of a tile of fewer queries the last wavefronts go without the last group)
    auto mine = [&](int g) { return g * 4 * kLineThreads + wave * 256 < tile; };

    // Finishes up to 64 of the `count` queries set aside, from the first-th on.
    auto finish = [&](uint32_t first, uint32_t count) {
        const bool have = first + (uint32_t)lane < count;
        const v4i e = l_open[have ? first + (uint32_t)lane : first];
        const uint32_t s = have ? (uint32_t)e.w : (uint32_t)tv.S, d = line_threshold(ix, e.z, acc_base_m1);
        const uint4 rh = tv.rank_hdr[s];
        const bool scan = have && rh.w != 0u;
        uint32_t plane;
        const uint32_t code = follow_lines(ix, have && !scan ? kCodeOpen : kCodeNone, s, d, (uint32_t)e.y, tv.S, plane);
        const bool hit = code < kCodeOpen;
        int32_t ans = hit ? (ix.line_rows() ? (int32_t)(code & row_mask) : ix.step_row[ix.hdr[s].z + (code & row_mask)]) : -1;
        st[1] += (uint32_t)__builtin_popcountll(__ballot(hit && plane > 1u));
        st[2] += (uint32_t)__builtin_popcountll(__ballot(hit && plane == 1u));
        const uint64_t scanned = __ballot(scan);
        if (scanned) {
            st[3] += (uint32_t)__builtin_popcountll(scanned);
            const uint4 none = make_uint4(0u, 0u, 0u, 0u);
            const int32_t row = ranked_first_fit<false>(tv, scan ? rh : none, e.z, (uint32_t)e.y);
            ans = scan ? row : ans;
        }
        st[4] += (uint32_t)__builtin_popcountll(__ballot(have && ans < 0));
        if (have && ans >= 0) q.out[e.x] = ans;   // (-1 is there)
    };
    auto finish_all = [&](uint32_t count) {   // the whole workgroup
        // another wavefront's stores for the same queries come first
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        for (uint32_t first = (uint32_t)wave * 64u; first < count; first += kLineThreads) finish(first, count);
        lds_barrier();
        if (tid == 0) l_count = 0u;
    };

    for (int64_t base = (int64_t)blockIdx.x * tile; base < q.n; base += (int64_t)gridDim.x * tile) {
        lds_barrier();
        const uint32_t waiting = l_count;
        if (waiting >= kLineDrain) finish_all(waiting);
        const bool whole = aligned && base + tile <= q.n;
        v4i f[4][kGroups];
        if (whole) {   // (every byte is used once: non-temporal)
#pragma unroll
            for (int g = 0; g < kGroups; ++g) {
                if (!mine(g)) continue;
                const int64_t i = base + g * 4 * kLineThreads + tid * 4;
                f[0][g] = __builtin_nontemporal_load((const v4i *)(q.task + i)); f[1][g] = __builtin_nontemporal_load((const v4i *)(q.slo + i));
                f[2][g] = __builtin_nontemporal_load((const v4i *)(q.min_acc + i)); f[3][g] = __builtin_nontemporal_load((const v4i *)(q.bidx + i));
            }
        } else {
#pragma unroll
            for (int g = 0; g < kGroups; ++g)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int64_t i = base + g * 4 * kLineThreads + tid * 4 + e;
                    const bool in = mine(g) && i < q.n;
                    f[0][g][e] = in ? q.task[i] : -1; f[1][g][e] = in ? q.slo[i] : -1;
                    f[2][g][e] = in ? q.min_acc[i] : 0; f[3][g][e] = in ? q.bidx[i] : -1;
                }
        }
        // the fields of the whole tile are there: from here on lines only.  (Waited for by name: a barrier alone leaves the waits to the compiler,
        // which puts them where a group's fields are used, and the phases run into each other: 64M queries 634 us instead of 453.)
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
        for (int g = 0; g < kGroups; ++g) {
            if (!mine(g)) continue;
            const int64_t i = base + g * 4 * kLineThreads + tid * 4;
            v4i r;
            uint64_t m[4];
            uint32_t total = 0, slice[4], thr[4], lim[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const uint32_t t = (uint32_t)f[0][g][e], b = (uint32_t)f[3][g][e];
                const bool ok = (t < (uint32_t)tv.T) & (b < (uint32_t)tv.B) & (f[1][g][e] >= 0);   // (others: the empty slice)
                slice[e] = ok ? t * (uint32_t)tv.B + b : (uint32_t)tv.S;
                thr[e] = line_threshold(ix, f[2][g][e], acc_base_m1);
                lim[e] = (uint32_t)f[1][g][e];
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const uint32_t code = lookup_lines<false>(ix.lines, slice[e] * kLineBytes, thr[e], lim[e], row_mask);
                r[e] = code < kCodeOpen ? (int32_t)(code & row_mask) : -1;
                m[e] = __ballot(code >= kCodeOpen && code < kCodeNone);
                total += (uint32_t)__builtin_popcountll(m[e]);
            }
            if (total) {
                uint32_t at = 0;
                if (lane == 0) at = atomicAdd(&l_count, total);
                at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if ((m[e] >> lane) & 1u) l_open[at + lanes_below(m[e])] = v4i{(int32_t)(i + e), (int32_t)lim[e], f[2][g][e], (int32_t)slice[e]};
                    at += (uint32_t)__builtin_popcountll(m[e]);
                }
                st[0] += total;
            }
            if (!ix.line_rows()) {   // entries name steps
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (r[e] >= 0) r[e] = ix.step_row[ix.hdr[slice[e]].z + (uint32_t)r[e]];
            }
            if (whole) {
                __builtin_nontemporal_store(r, (v4i *)(q.out + i));
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (i + e < q.n) q.out[i + e] = r[e];
            }
        }
    }
    lds_barrier();
    const uint32_t waiting = l_count;
    if (waiting) finish_all(waiting);
    if (lane == 0) {
#pragma unroll
        for (int k = 0; k < kLookupStats; ++k)
            if (st[k]) atomicAdd(&l_st[k], st[k]);
    }
    __syncthreads();
    if (tid < kLookupStats) ix.stats[blockIdx.x * kLookupStats + tid] = l_st[tid];
    if (blockIdx.x == 0 && tid == 0) ix.stats[-1] = gridDim.x;
}

}  // namespace

// ---------------------------------------------------------------- launcher

hipError_t launch_line_select(const TableView &tv, const IndexView &ix, const QueryView &q, int num_cus, hipStream_t st,
                              const LaunchEvents *ev)
{
    // the same share for every workgroup, in as many tiles as it takes (2.5M queries on 8000 slices: 35 us with full tiles, of which
    // every sixth workgroup has two, 28 so)
    const int64_t most = (int64_t)kLineThreads * kLineQueries, turns = ((int64_t)q.n + most * num_cus - 1) / (most * num_cus);
    const int64_t tile = (((int64_t)q.n + turns * num_cus - 1) / (turns * num_cus) + 255) & ~255ll, tiles = ((int64_t)q.n + tile - 1) / tile;
    const hipError_t e = hipFuncSetAttribute((const void *)k_line_select, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLineOpenLds);
    if (e != hipSuccess) return e;
    return launch_kernel(ev, k_line_select, dim3((unsigned)(tiles < num_cus ? tiles : num_cus)), dim3(kLineThreads), kLineOpenLds, st, tv, ix, q, (int32_t)tile);
}

}  // namespace infaas
