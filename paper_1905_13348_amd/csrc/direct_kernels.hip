// The selection (Section 4.1 of the INFaaS paper) straight from global memory, one lane per query: no LDS
// mirror to fill, no queues, as many wavefronts in flight as the queries give.
#include "internal.h"
#include "lookup_common.h"

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
    const int64_t at = in ? i : 0;   // (every lane reads: four loads in a row, without branches; there is a query 0)
    u.task = q.task[at]; u.slo = q.slo[at]; u.min_acc = q.min_acc[at]; u.bidx = q.bidx[at];
    u.task = in ? u.task : -1;
    u.inside = (uint32_t)u.task < (uint32_t)tv.T && (uint32_t)u.bidx < (uint32_t)tv.B;
    u.valid = u.inside && u.slo >= 0;
    u.s = u.inside ? (uint32_t)u.task * (uint32_t)tv.B + (uint32_t)u.bidx : (uint32_t)tv.S;
    return u;
}

// The selection for the lanes in `want` (of valid queries), -1 elsewhere.  `rounds`: of lookup_lines, those of the lanes that have
// queries at all.  kRanked: slices that the index does not hold completely go through their entries in rank order at once;
// otherwise only with what their lines leave open.  Counts in st what became of the queries; there is no mirror, so all of
// them count as set aside.
// incomplete: there are such slices, and their queries do so here too.
template <bool kRanked, bool kAhead>
__device__ __forceinline__ int32_t select_from_memory(const TableView &tv, const IndexView &ix, const Query &u, bool want, uint32_t rounds, bool packed, bool incomplete,
                                                      uint32_t (&st)[kLookupStats])
{
    auto count = [&](int what, bool yes) { st[what] += (uint32_t)__builtin_popcountll(__ballot(yes)); };
    uint32_t s = want ? u.s : (uint32_t)tv.S;
    uint4 rh{};
    bool scan = false;
    if (kRanked || incomplete) {
        rh = tv.rank_hdr[s];
        scan = want && rh.w != 0u;
        s = scan ? (uint32_t)tv.S : s;
    }
    int32_t ans = -1;
    if (!kRanked || __ballot(want && !scan)) {
        const uint32_t d = line_threshold(ix, u.min_acc, tv.acc_base - 1), l = (uint32_t)u.slo, row_mask = (1u << ix.line_shift()) - 1u;
        uint32_t code, plane;
        if (packed) code = lookup_lines_packed(ix.lines, __ballot(want), s * kLineBytes, d, l, row_mask);
        else if (rounds == 15u) code = lookup_lines<false>(ix.lines, s * kLineBytes, d, l, row_mask);
        else code = lookup_lines<true>(ix.lines, s * kLineBytes, d, l, row_mask, rounds);
        code = want ? code : kCodeNone;   // (of a round that was left out: nothing)
        code = follow_lines(ix, code, s, d, l, tv.S, plane);
        const bool hit = code < kCodeOpen;
        if (hit) ans = ix.line_rows() ? (int32_t)(code & row_mask) : ix.step_row[ix.hdr[s].z + (code & row_mask)];
        if (!kRanked) scan = scan || code == kCodeRank;
        count(1, hit && plane > 1u);
        count(2, hit && plane <= 1u);
    }
    if (__ballot(scan)) {
        if (!kRanked && !incomplete) rh = tv.rank_hdr[s];
        const int32_t row = ranked_first_fit<kAhead>(tv, scan ? rh : make_uint4(0u, 0u, 0u, 0u), u.min_acc, (uint32_t)u.slo);
        if (scan) ans = row;
        count(3, scan);
    }
    count(0, want);
    count(4, want && ans < 0);
    return ans;
}

// The closest variant of the table for the lanes in `want` (queries inside the table that nothing satisfies),
// and how far it is from the requirements: from the lines, or where they do not hold all of the slice's steps
// by the wavefront over the whole slice.
__device__ __forceinline__ int32_t closest_from_memory(const TableView &tv, const IndexView &ix, const Query &u, bool want, bool incomplete, HowFar &how)
{
    const uint32_t s = want ? u.s : (uint32_t)tv.S;
    const bool scan = incomplete && tv.rank_hdr[s].w != 0u;
    uint32_t code = closest_in_lines(ix, want && !scan, s, tv.S, line_threshold(ix, u.min_acc, tv.acc_base - 1), u.slo, u.min_acc, tv.acc_base - 1, how);
    code = scan ? kCodeRank : code;
    int32_t sug = -1;
    if (want && code < kCodeOpen) sug = ix.line_rows() ? (int32_t)code : ix.step_row[ix.hdr[s].z + code];
    uint64_t rest = __ballot(want && code == kCodeRank);
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

// The workgroup's counts into its entry of the statistics.
__device__ __forceinline__ void leave_statistics(const IndexView &ix, const uint32_t (&st)[kLookupStats])
{
    __shared__ uint32_t l_st[kDirThreads / 64][kLookupStats];
    if ((threadIdx.x & 63) == 0) {
#pragma unroll
        for (int k = 0; k < kLookupStats; ++k) l_st[threadIdx.x >> 6][k] = st[k];
    }
    __syncthreads();
    if (threadIdx.x < kLookupStats) {
        uint32_t sum = 0;
#pragma unroll
        for (int w = 0; w < kDirThreads / 64; ++w) sum += l_st[w][threadIdx.x];
        ix.stats[blockIdx.x * kLookupStats + threadIdx.x] = sum;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) ix.stats[-1] = gridDim.x;
}

// Where the lanes' queries are: `per` of them to a wavefront, so that few of them are spread over its quads, each of which
// reads one line at a time.
struct Spread {
    int32_t number;   // of this lane's query
    bool mine;        // it has one
    uint32_t rounds;  // of lookup_lines, those of the lanes that have
};
__device__ __forceinline__ Spread spread_of(int32_t spread)   // 2^spread lanes to a query
{
    const int32_t lane = threadIdx.x & 63;
    return Spread{lane >> spread, (lane & ((1 << spread) - 1)) == 0, spread == 0 ? 15u : spread == 1 ? 5u : 1u};
}

// Bound by the rate of scattered reads, a line (4.5 ps) and its share of further ones per query, and below 100,000 queries by the launch
// and three dependent trips to memory (arguments, fields, line).
template <bool kRanked>
__global__ __launch_bounds__(kDirThreads) void k_direct_select(TableView tv, IndexView ix, QueryView q, int32_t spread)
{
    const int32_t wave = threadIdx.x >> 6, per = 64 >> spread, step = per * (kDirThreads / 64);
    const Spread sp = spread_of(spread);
    const uint32_t news = request_index_stats(tv);
    bool first = true;
    uint32_t st[kLookupStats] = {0u, 0u, 0u, 0u, 0u};
    for (int64_t i0 = (int64_t)blockIdx.x * step; i0 < q.n; i0 += (int64_t)gridDim.x * step) {
        const int64_t i = i0 + wave * per + sp.number;
        const Query u = load_query(tv, q, i, sp.mine);
        if (first) hand_on_index_stats(tv, news);
        first = false;
        const int32_t ans = select_from_memory<kRanked, true>(tv, ix, u, u.valid, sp.rounds, false, false, st);
        if (sp.mine && i < q.n) q.out[i] = ans;
    }
    leave_statistics(ix, st);
}

// The other modes of the lookup in one launch: both tiers after one another for the lanes that need them, no lists
// in between.  kTiers: ta / ia serve the Active variants, tb / ib the Inactive ones (otherwise there is only ta);
// kSuggest: the closest variant (of both tiers) where there is no answer; kWorker: the worker of every answer.
// Bound by its launch and the chain of dependent reads, like the two passes of the lookup kernel that it replaces, but
// once and without the two LDS mirrors.
template <bool kTiers, bool kSuggest, bool kWorker>
__global__ __launch_bounds__(kDirThreads) void k_direct_modes(TableView ta, IndexView ia, TableView tb, IndexView ib, QueryView q, int32_t spread, bool incomplete)
{
    const int32_t per = 64 >> spread, step = per * (kDirThreads / 64);
    const Spread sp = spread_of(spread);
    const uint32_t news = request_index_stats(ta), news2 = kTiers ? request_index_stats(tb) : 0u;
    bool first = true;
    uint32_t st[kLookupStats] = {0u, 0u, 0u, 0u, 0u};
    for (int64_t i0 = (int64_t)blockIdx.x * step; i0 < q.n; i0 += (int64_t)gridDim.x * step) {
        const int64_t i = i0 + (int32_t)(threadIdx.x >> 6) * per + sp.number;
        const bool mine = sp.mine;
        const Query u = load_query(ta, q, i, mine);
        if (first) hand_on_index_stats(ta, news);
        if (kTiers && first) hand_on_index_stats(tb, news2);
        first = false;
        int32_t ans = select_from_memory<false, false>(ta, ia, u, u.valid, sp.rounds, false, incomplete, st), tier = ans >= 0 ? 1 : 0;
        if (kTiers) {
            const bool next = u.valid && ans < 0;
            if (__ballot(next)) {
                const int32_t row = select_from_memory<false, false>(tb, ib, u, next, 15u, __builtin_popcountll(__ballot(next)) <= 48, incomplete, st);
                if (next && row >= 0) { ans = row; tier = 2; }
            }
        }
        int32_t closest = ans;
        if (kSuggest) {
            const bool none = u.inside && ans < 0;
            if (__ballot(none)) {
                HowFar how;
                int32_t sug = closest_from_memory(ta, ia, u, none, incomplete, how);
                if (kTiers) {   // the closer of the two tiers' suggestions, the first tier's at a tie
                    HowFar how2;
                    const int32_t sug2 = closest_from_memory(tb, ib, u, none, incomplete, how2);
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
    leave_statistics(kTiers ? ib : ia, st);
}

// How many queries a wavefront takes.  A batch too small to give every SIMD two full wavefronts is spread over as many with fewer queries
// each, down to the 16 that are one round of lookup_lines.  In rank order, where a
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

hipError_t launch_direct_select(const TableView &tv, const IndexView &ix, const QueryView &q, bool ranked, int num_cus,
                                hipStream_t st, const LaunchEvents *ev)
{
    const int32_t per = queries_per_wave(q.n, ranked ? 1 : 16, num_cus);
    const int64_t step = per * (kDirThreads / 64), want = ((int64_t)q.n + step - 1) / step, most = index_stat_blocks(num_cus);
    auto kernel = ranked ? k_direct_select<true> : k_direct_select<false>;
    return launch_kernel(ev, kernel, dim3((unsigned)(want < most ? want : most)), dim3(kDirThreads), 0, st, tv, ix, q, __builtin_ctz(64u / (unsigned)per));
}

hipError_t launch_direct_modes(const TableView &ta, const IndexView &ia, const TableView &tb, const IndexView &ib, const QueryView &q,
                               bool tiers, bool incomplete, int num_cus, hipStream_t st, const LaunchEvents *ev)
{
    const int32_t per = queries_per_wave(q.n, 16, num_cus);
    const int64_t step = per * (kDirThreads / 64), want = ((int64_t)q.n + step - 1) / step, most = index_stat_blocks(num_cus);
    auto kernel = !tiers ? k_direct_modes<false, true, false> : q.worker ? (q.closest ? k_direct_modes<true, true, true> : k_direct_modes<true, false, true>)
                                                              : (q.closest ? k_direct_modes<true, true, false> : k_direct_modes<true, false, false>);
    return launch_kernel(ev, kernel, dim3((unsigned)(want < most ? want : most)), dim3(kDirThreads), 0, st, ta, ia, tb, ib, q, __builtin_ctz(64u / (unsigned)per), incomplete);
}

}  // namespace infaas
