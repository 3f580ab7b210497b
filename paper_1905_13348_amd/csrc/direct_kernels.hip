// The selection (Section 4.1 of the INFaaS paper) straight from global memory, one lane per query: no LDS
// mirror to fill, no queues, as many wavefronts in flight as the queries give.
#include "internal.h"
#include "lookup_common.h"

#include <type_traits>

namespace infaas {

namespace {

constexpr int kDirThreads = 256;

// The slice of one query per lane and what the lookups of all modes need of it.
struct Query {
    int32_t task, bidx, slo, min_acc;
    bool inside, valid;   // names a slice of the table; and has a bound that anything can meet
    uint32_t s;           // its slice, or the empty one
};
__device__ __forceinline__ Query load_query(const TableView &tv, const QueryView &q, int64_t i, bool mine = true)
{
    const bool in = mine && i < q.n;
    Query u;
    u.task = in ? q.task[i] : -1; u.slo = in ? q.slo[i] : -1; u.min_acc = in ? q.min_acc[i] : 0; u.bidx = in ? q.bidx[i] : -1;
    u.inside = (uint32_t)u.task < (uint32_t)tv.T && (uint32_t)u.bidx < (uint32_t)tv.B;
    u.valid = u.inside && u.slo >= 0;
    u.s = u.inside ? (uint32_t)u.task * (uint32_t)tv.B + (uint32_t)u.bidx : (uint32_t)tv.S;
    return u;
}

// The selection for the lanes in `want` (of valid queries), -1 elsewhere.  kRanked: slices whose steps are not all
// in their bodies go through their entries in rank order at once; otherwise only with what the bodies leave
// open.  Counts in st what became of the queries, as the lookup kernel does; no query is decided by an
// LDS copy here, so all count as parked.
template <bool kRanked, bool kAhead, bool kByFour>
__device__ __forceinline__ int32_t select_from_memory(const TableView &tv, const IndexView &ix, const Query &u, bool want,
                                                      uint32_t (&st)[kLookupStats])
{
    auto count = [&](int what, bool yes) { st[what] += (uint32_t)__builtin_popcountll(__ballot(yes)); };
    int nit = 0;
    if (!kByFour) nit = 32 - __builtin_clz(ix.ctrl[kCtlMaxK0] | 1u);    // <= 5
    const uint32_t s = want ? u.s : (uint32_t)tv.S;
    const uint4 h = ix.hdr[s];
    uint4 rh{};
    if (kRanked) rh = tv.rank_hdr[s];
    int32_t ans = -1;
    const bool body = want && !(h.y & kHdrPark) && !(kRanked && (h.y & kHdrTrunc));
    if (__ballot(body)) {
        const uint32_t keys0 = (h.y >> kHdrK0Shift) & 0x3Fu, keys1 = (h.y >> kHdrK1Shift) & 0x3Fu;
        const uint32_t dd = acc_threshold(u.min_acc, tv.acc_base - 1), lim = (uint32_t)u.slo;
        uint32_t m = 0u;
        auto search = [&](bool on, uint32_t at, uint32_t re) __attribute__((always_inline)) {
            if constexpr (kByFour) {
                const uint32_t a = on ? at : 0u, r = on ? re : 0u;
                if ((__ballot(on) >> 32) == 0ull) search_bodies_by_four<1>(ix.pool, a, r, dd, lim, m);
                else search_bodies_by_four<4>(ix.pool, a, r, dd, lim, m);
            } else {
                const uint32_t a1[1] = {on ? at : 0u}, r1[1] = {on ? re : 2u}, d1[1] = {dd}, l1[1] = {lim};
                uint32_t m1[1];
                search_bodies<1>(GlobalMem{ix.pool}, nit, a1, r1, d1, l1, m1);
                m = on ? m1[0] : 0u;
            }
        };
        search(body, h.x, keys0);
        const bool hit0 = m != 0u;
        uint32_t at = hit0 ? h.z + (uint32_t)__builtin_ctz(m) : 0u;   // (entry 0 of step_row is -1)
        count(2, hit0);
        const bool more = body && !hit0 && keys1 != 0u;
        if (__ballot(more)) {
            search(more, h.x + body_bytes(keys0), keys1);
            const bool hit1 = m != 0u;
            if (hit1) at = h.z + kBodySteps + (uint32_t)__builtin_ctz(m);
            count(1, hit1);
        }
        ans = ix.step_row[at];
    }
    const bool scan = want && ans < 0 && (h.y & kHdrTrunc);
    if (__ballot(scan)) {
        if (!kRanked) rh = tv.rank_hdr[s];
        const int32_t row = ranked_first_fit<kAhead>(tv, scan ? rh : make_uint4(0u, 0u, 0u, 0u), u.min_acc, (uint32_t)u.slo);
        if (scan) ans = row;
        count(3, scan);
    }
    count(0, want);
    count(4, want && ans < 0);
    return ans;
}

// The closest variant of the table for the lanes in `want` (queries inside the table that nothing satisfies),
// and how far it is from the requirements: from the bodies, or where they are not all of the slice's steps
// by the wavefront over the whole slice.
__device__ __forceinline__ int32_t closest_from_memory(const TableView &tv, const IndexView &ix, const Query &u, bool want, HowFar &how)
{
    how = HowFar{3, 0, 0};
    int32_t sug = -1;
    const uint32_t s = want ? u.s : (uint32_t)tv.S;
    const uint4 h = ix.hdr[s];
    const bool by_index = want && !(h.y & (kHdrPark | kHdrTrunc));
    if (__ballot(by_index)) {
        const uint32_t max_k = ix.ctrl[kCtlMaxK0];
        const ClosestStep c = closest_step(GlobalMem{ix.pool}, 32 - __builtin_clz(max_k | 1u), by_index ? h.x : 0u,
                                           by_index ? (h.y >> kHdrK0Shift) & 0x3Fu : 2u, by_index ? (h.y >> kHdrK1Shift) & 0x3Fu : 0u,
                                           acc_threshold(u.min_acc, tv.acc_base - 1), u.slo, u.min_acc, tv.acc_base - 1);
        if (by_index && c.step >= 0) { sug = ix.step_row[h.z + (uint32_t)c.step]; how = c.how; }
    }
    uint64_t rest = __ballot(want && !by_index);
    while (rest) {
        const int l = __builtin_ctzll(rest);
        rest &= rest - 1;
        HowFar far;
        const int32_t found = closest_by_scan(tv, __builtin_amdgcn_readlane(u.task, l), __builtin_amdgcn_readlane(u.bidx, l),
                                              __builtin_amdgcn_readlane(u.min_acc, l), __builtin_amdgcn_readlane(u.slo, l),
                                              (int)(threadIdx.x & 63), &far);
        if ((int)(threadIdx.x & 63) == l) { sug = found; how = far; }
    }
    return sug;
}

// The workgroup's counts into its entry of the statistics (l_st: kLookupStats words of LDS, cleared before).
__device__ __forceinline__ void leave_statistics(const IndexView &ix, uint32_t *l_st, const uint32_t (&st)[kLookupStats])
{
    if ((threadIdx.x & 63) == 0) {
#pragma unroll
        for (int k = 0; k < kLookupStats; ++k)
            if (st[k]) atomicAdd(&l_st[k], st[k]);
    }
    __syncthreads();
    if (threadIdx.x < kLookupStats) ix.stats[blockIdx.x * kLookupStats + threadIdx.x] = l_st[threadIdx.x];
    if (blockIdx.x == 0 && threadIdx.x == 0) ix.stats[-1] = gridDim.x;
}

// Bound by the rate of scattered reads (header, three to five lines of the body, two sets, row: 20 ps per query, 40 with the lane's
// own bisection, which kByFour false keeps for bodies that L1 holds).  The lanes of a wavefront take `per` queries.
template <bool kRanked, bool kByFour>
__global__ __launch_bounds__(kDirThreads) void k_direct_select(TableView tv, IndexView ix, QueryView q, int32_t per)
{
    const int32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6, step = per * (kDirThreads / 64);
    __shared__ uint32_t l_st[kLookupStats];
    publish_index_stats(tv);
    if (threadIdx.x < kLookupStats) l_st[threadIdx.x] = 0u;
    __syncthreads();
    uint32_t st[kLookupStats] = {0u, 0u, 0u, 0u, 0u};
    for (int64_t i0 = (int64_t)blockIdx.x * step; i0 < q.n; i0 += (int64_t)gridDim.x * step) {
        const int64_t i = i0 + wave * per + lane;
        const bool mine = lane < per;
        const Query u = load_query(tv, q, i, mine);
        const int32_t ans = select_from_memory<kRanked, true, kByFour>(tv, ix, u, u.valid, st);
        if (mine && i < q.n) q.out[i] = ans;
    }
    leave_statistics(ix, l_st, st);
}

// The other modes of the lookup in one launch: both tiers after one another for the lanes that need them, no lists
// in between.  kTiers: ta / ia serve the Active variants, tb / ib the Inactive ones (otherwise there is only ta);
// kSuggest: the closest variant (of both tiers) where there is no answer; kWorker: the worker of every answer.
// Bound by its launch and the chain of dependent reads, like the two passes of the lookup kernel that it replaces, but
// once and without the two LDS mirrors.
template <bool kTiers, bool kSuggest, bool kWorker, bool kByFour>
__global__ __launch_bounds__(kDirThreads) void k_direct_modes(TableView ta, IndexView ia, TableView tb, IndexView ib, QueryView q, int32_t per)
{
    const int32_t lane = threadIdx.x & 63, step = per * (kDirThreads / 64);
    __shared__ uint32_t l_st[kLookupStats];
    publish_index_stats(ta);
    if (kTiers) publish_index_stats(tb);
    if (threadIdx.x < kLookupStats) l_st[threadIdx.x] = 0u;
    __syncthreads();
    uint32_t st[kLookupStats] = {0u, 0u, 0u, 0u, 0u};
    for (int64_t i0 = (int64_t)blockIdx.x * step; i0 < q.n; i0 += (int64_t)gridDim.x * step) {
        const int64_t i = i0 + (int32_t)(threadIdx.x >> 6) * per + lane;
        const bool mine = lane < per;
        const Query u = load_query(ta, q, i, mine);
        int32_t ans = select_from_memory<false, false, kByFour>(ta, ia, u, u.valid, st), tier = ans >= 0 ? 1 : 0;
        if (kTiers) {
            const bool next = u.valid && ans < 0;
            if (__ballot(next)) {
                const int32_t row = select_from_memory<false, false, kByFour>(tb, ib, u, next, st);
                if (next && row >= 0) { ans = row; tier = 2; }
            }
        }
        int32_t closest = ans;
        if (kSuggest) {
            const bool none = u.inside && ans < 0;
            if (__ballot(none)) {
                HowFar how;
                int32_t sug = closest_from_memory(ta, ia, u, none, how);
                if (kTiers) {   // the closer of the two tiers' suggestions, the first tier's at a tie
                    HowFar how2;
                    const int32_t sug2 = closest_from_memory(tb, ib, u, none, how2);
                    if (sug2 >= 0 && !(sug >= 0 && closer_or_equal(how, how2))) sug = sug2;
                }
                if (none) closest = sug;
            }
        }
        if (mine && i < q.n) {
            q.out[i] = ans;
            if (kTiers) q.tier[i] = tier;
            if (kSuggest) q.closest[i] = closest;
            if (kWorker) q.worker[i] = ans >= 0 ? q.row_worker[(tier == 2 ? ta.V : 0) + ans] : -1;
        }
    }
    leave_statistics(kTiers ? ib : ia, l_st, st);
}

// Who searches a body: its lane by bisection, which is fast where L1 holds the lines that it probes, or four lanes that read all of its
// keys (search_bodies_by_four), which takes a third more registers and more instructions.  Kernel us, bisection / four lanes, by the bytes of
// the bodies:
//   selection, 100,000 queries: 5 KB 4.2 / 4.6, 23 KB 5.2 / 5.4, 38 KB 5.1 / 5.0, 42 KB (two bodies to a slice) 5.8 / 6.4, 62 KB 5.6 / 5.5,
//     92 KB 5.5 / 4.8, 134 KB 6.0 / 5.4, 173 KB 6.9 / 4.9
//   two tiers, 1001 / 100,000 / 200,000: 5 KB 6.0 / 6.5 / 8.4 and 5.9 / 7.6 / 9.9, 38 KB 6.3 / 6.5 / 9.9 and 6.1 / 6.9 / 10.3, 60 KB 5.0 / 6.4 / 9.0
//     and 4.8 / 7.0 / 9.5, 92 KB 5.4 / 7.0 / 10.5 and 4.9 / 7.0 / 9.4, 173 KB 6.7 / 8.6 / 13.1 and 6.4 / 8.0 / 10.9
//   with a suggestion, one table, 60,000 / 80,000: 5 KB 7.2 / 7.7 and 7.7 / 8.5, 62 KB 7.4 / 8.4 and 7.7 / 8.4, 92 KB 7.4 / 8.2 and 7.6 / 8.0, 173 KB
//     9.1 / 10.0 and 8.8 / 9.4
//   and two tiers, 45,000 / 100,000 / 200,000: 5 KB 11.4 / 12.0 / 14.8 and 12.7 / 13.6 / 17.1, 62 KB 11.8 / 13.0 / 16.0 and 12.4 / 13.8 / 16.8,
//     92 KB 11.8 / 13.3 / 16.6 and 12.5 / 14.2 / 16.9, 134 KB 12.0 / 13.7 / 17.9 and 12.8 / 14.4 / 17.2, 250 KB 12.6 / 14.6 / 20.4 and 13.6 / 15.0 / 18.3
bool four_lanes(bool tiers, bool suggest, int64_t n, int32_t per, int64_t pool, int num_cus)
{
    if (!tiers && !suggest) return pool > 48 * 1024;
    if (!suggest) return per == 16 || pool > 64 * 1024;
    return tiers ? n > (int64_t)num_cus * 512 && pool > 96 * 1024 : per == 64 && pool > 64 * 1024;
}

// How many queries a wavefront takes.  A batch too small to give every SIMD two full wavefronts is spread over as many with fewer queries
// each, down to the 16 that one round of search_bodies_by_four serves (two tiers, 1001 queries 8.5 -> 6.6 us, with workers 8.6 -> 6.7; to
// bisection 16 to 64 of them are the same in a selection, and 16 up to 7% faster with two tiers).  In rank order, where a
// wavefront finishes its hard queries one after the other, down to one.  (us for 1001 / 10,001 / 30,001 queries, 64 to a wavefront and so: 2000 entries of random
// accuracy and latency to a slice, most queries without an answer, 75 / 75 / 76 and 6.1 / 14 / 23, with the scan engine 37 / 63 / 89; every entry a step, nothing
// hard about it, 6.0 / 6.1 / 6.1 and 6.2 / 6.2 / 6.2, where four wavefronts per SIMD took 6.1 / 6.6 / 8.1.)
int32_t queries_per_wave(int64_t n, int32_t least, int num_cus)
{
    int32_t per = 64;
    while (per > least && (n + per / 2 - 1) / (per / 2) <= (int64_t)num_cus * 8) per /= 2;
    return per;
}

}  // namespace

hipError_t launch_direct_select(const TableView &tv, const IndexView &ix, const QueryView &q, bool ranked, int64_t pool, int num_cus,
                                hipStream_t st, const LaunchEvents *ev)
{
    const int32_t per = queries_per_wave(q.n, ranked ? 1 : 16, num_cus);
    const int64_t step = per * (kDirThreads / 64), want = ((int64_t)q.n + step - 1) / step, most = index_stat_blocks(num_cus);
    auto kernel = ranked ? k_direct_select<true, true> : four_lanes(false, false, q.n, per, pool, num_cus) ? k_direct_select<false, true> : k_direct_select<false, false>;
    return launch_kernel(ev, kernel, dim3((unsigned)(want < most ? want : most)), dim3(kDirThreads), 0, st, tv, ix, q, per);
}

hipError_t launch_direct_modes(const TableView &ta, const IndexView &ia, const TableView &tb, const IndexView &ib, const QueryView &q,
                               bool tiers, int64_t pool, int num_cus, hipStream_t st, const LaunchEvents *ev)
{
    const int32_t per = queries_per_wave(q.n, 16, num_cus);
    const int64_t step = per * (kDirThreads / 64), want = ((int64_t)q.n + step - 1) / step, most = index_stat_blocks(num_cus);
    auto pick = [&](auto by_four) {
        constexpr bool f = decltype(by_four)::value;
        return !tiers ? k_direct_modes<false, true, false, f> : q.worker ? (q.closest ? k_direct_modes<true, true, true, f> : k_direct_modes<true, false, true, f>)
                                                              : (q.closest ? k_direct_modes<true, true, false, f> : k_direct_modes<true, false, false, f>);
    };
    auto kernel = four_lanes(tiers, q.closest != nullptr, q.n, per, pool, num_cus) ? pick(std::true_type{}) : pick(std::false_type{});
    return launch_kernel(ev, kernel, dim3((unsigned)(want < most ? want : most)), dim3(kDirThreads), 0, st, ta, ia, tb, ib, q, per);
}

}  // namespace infaas
