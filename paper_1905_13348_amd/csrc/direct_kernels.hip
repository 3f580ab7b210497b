// The selection (Section 4.1 of the INFaaS paper) straight from global memory, one lane per query: no LDS
// mirror to fill, no queues, as many wavefronts in flight as the queries give.
#include "internal.h"
#include "lookup_common.h"

namespace infaas {

namespace {

constexpr int kDirThreads = 256;

// kRanked: slices whose steps are not all in their bodies go through their entries in rank order at once (for
// tables that consist mostly of such slices); otherwise only with what the bodies leave open.
// Bound by the rate of scattered reads: 14 per query through a body (header, ten probes, two sets, row), each
// lane another line.  Sixteen wavefronts per compute unit already saturate that: register caps for 24 to 32
// (80 to 64 registers instead of 89) were measured 0-25% slower on batches of a million.
template <bool kRanked>
__global__ __launch_bounds__(kDirThreads) void k_direct_select(TableView tv, IndexView ix, QueryView q)
{
    __shared__ uint32_t l_st[kLookupStats];
    const int tid = threadIdx.x, lane = tid & 63;
    publish_index_stats(tv);
    if (tid < kLookupStats) l_st[tid] = 0u;
    __syncthreads();
    const int32_t acc_base_m1 = tv.acc_base - 1;
    const uint32_t max_k = ix.ctrl[kCtlMaxK0];
    const int nit = 32 - __builtin_clz(max_k | 1u);    // <= 5
    const GlobalMem gmem{ix.pool};
    // as in the lookup kernel; no query is decided by an LDS copy here, so all valid ones count as parked
    uint32_t st[kLookupStats] = {0u, 0u, 0u, 0u, 0u};
    auto count = [&](int what, bool yes) { st[what] += (uint32_t)__builtin_popcountll(__ballot(yes)); };
    for (int64_t i0 = (int64_t)blockIdx.x * kDirThreads + (tid & ~63); i0 < q.n; i0 += (int64_t)gridDim.x * kDirThreads) {
        const int64_t i = i0 + lane;
        const bool in = i < q.n;
        const int32_t task = in ? q.task[i] : -1, slo = in ? q.slo[i] : -1, min_acc = in ? q.min_acc[i] : 0;
        const int32_t bidx = in ? q.bidx[i] : -1;
        const bool valid = (uint32_t)task < (uint32_t)tv.T && (uint32_t)bidx < (uint32_t)tv.B && slo >= 0;
        const uint32_t s = valid ? (uint32_t)task * (uint32_t)tv.B + (uint32_t)bidx : (uint32_t)tv.S;
        const uint4 h = ix.hdr[s], rh = tv.rank_hdr[s];
        int32_t ans = -1;
        const bool body = valid && !(h.y & kHdrPark) && !(kRanked && (h.y & kHdrTrunc));
        if (__ballot(body)) {
            const uint32_t keys0 = (h.y >> kHdrK0Shift) & 0x3Fu, keys1 = (h.y >> kHdrK1Shift) & 0x3Fu;
            const uint32_t dd[1] = {acc_threshold(min_acc, acc_base_m1)}, lim[1] = {(uint32_t)slo};
            const uint32_t bd[1] = {body ? h.x : 0u}, ks[1] = {body ? keys0 : 2u};
            uint32_t m[1];
            search_bodies<1>(gmem, nit, bd, ks, dd, lim, m);
            const bool hit0 = body && m[0] != 0u;
            uint32_t at = hit0 ? h.z + (uint32_t)__builtin_ctz(m[0]) : 0u;   // (entry 0 of step_row is -1)
            count(2, hit0);
            const bool more = body && !hit0 && keys1 != 0u;
            if (__ballot(more)) {
                const uint32_t bd1[1] = {more ? h.x + body_bytes(keys0) : 0u}, ks1[1] = {more ? keys1 : 2u};
                search_bodies<1>(gmem, nit, bd1, ks1, dd, lim, m);
                const bool hit1 = more && m[0] != 0u;
                if (hit1) at = h.z + kBodySteps + (uint32_t)__builtin_ctz(m[0]);
                count(1, hit1);
            }
            ans = ix.step_row[at];
        }
        const bool scan = valid && ans < 0 && (h.y & kHdrTrunc);
        if (__ballot(scan)) {
            const int32_t row = ranked_first_fit(tv, scan ? rh : make_uint4(0u, 0u, 0u, 0u), min_acc, (uint32_t)slo);
            if (scan) ans = row;
            count(3, scan);
        }
        count(0, valid);
        count(4, valid && ans < 0);
        if (in) q.out[i] = ans;
    }
    if (lane == 0) {
#pragma unroll
        for (int k = 0; k < kLookupStats; ++k)
            if (st[k]) atomicAdd(&l_st[k], st[k]);
    }
    __syncthreads();
    if (tid < kLookupStats) ix.stats[blockIdx.x * kLookupStats + tid] = l_st[tid];
    if (blockIdx.x == 0 && tid == 0) *ix.stat_used = gridDim.x;
}

}  // namespace

hipError_t launch_direct_select(const TableView &tv, const IndexView &ix, const QueryView &q, bool ranked, int num_cus,
                                hipStream_t st, const LaunchEvents *ev)
{
    const int64_t want = ((int64_t)q.n + kDirThreads - 1) / kDirThreads, most = index_stat_blocks(num_cus);
    return launch_kernel(ev, ranked ? k_direct_select<true> : k_direct_select<false>, dim3((unsigned)(want < most ? want : most)), dim3(kDirThreads), 0, st, tv, ix, q);
}

}  // namespace infaas
