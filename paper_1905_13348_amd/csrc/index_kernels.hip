// Staircase index of the variant selection (Section 4.1 of the INFaaS paper): the same
// answers as the exhaustive scan, reached through a per-slice structure that keeps only the
// variants that can ever be chosen.  The paper's own controller answers in milliseconds where
// its brute-force search needs ~100 ms because its metadata store keeps sorted sets
// (Sections 5 and 6.4); this is the exact, batched GPU counterpart of that idea.
//
//   k_index_build  : one wavefront per (task, batch) slice finds the "steps" (variants that no
//                    cheaper one dominates), in rounds over a shrinking list of candidates, then
//                    writes sorted keys and bit sets for them (layout: internal.h)
//   k_index_select : one lane per query.  The whole index is mirrored in LDS; a query costs two
//                    5-probe binary searches in LDS, two bit-set reads, one AND and one count-
//                    trailing-zeros.  Queries the first body of their slice cannot decide (no
//                    fitting step among its first 31, slice not resident, staircase truncated)
//                    are parked in a queue of the wavefront and finished by it, 64 at a time or
//                    when it runs out of work: second body, index copy in global memory, and last
//                    a wavefront-wide scan of the rank-ordered slice that stops at the first
//                    feasible variant.  In its closest-variant mode the kernel also parks the
//                    queries that end without a feasible variant and finds, in the same bodies,
//                    the variant that comes closest to their requirements.
#include "internal.h"
#include "lookup_common.h"

#include <type_traits>

namespace infaas {

namespace {

constexpr int kSelThreads = 1024;
constexpr int kPerThread = 4;   // queries per lane and unit, searched interleaved (8 does not fit in 128 VGPRs)
constexpr uint32_t kParkFinal = 1u << 31;          // in a parked record's slice word: the selection is known to be -1
constexpr int kWaveQueue = 64 + 64 * kPerThread;   // parked queries a wavefront can hold: a full pass plus one unit

// ---------------------------------------------------------------- build

// Orders the LDS traffic of ONE wavefront: what its lanes have written is visible to its other lanes.
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}


// Body of steps [g0, g0 + kb), held one per lane (lanes g0..g0+kb-1), in two parts: what can be
// computed before the body's place in the pool is known, and the stores.
struct BodyRegs {
    int32_t pa, ps;     // position of this lane's step in the sorted accuracy / latency keys
    uint32_t ma, ms;    // lane p: A[p] and S[p], the steps among the p most accurate / p fastest
};
// Steps [g0, g0 + kb) of a slice: lane j holds step j in (st_acc, st_tot), and p_acc / p_tot hold all
// steps in LDS.  `ranks` is scratch of the wavefront (2 x 64 words).  Values that all lanes need are
// read from LDS (one address for all lanes), so the loops are plain vector code.
__device__ __forceinline__ BodyRegs body_compute(int g0, int kb, int lane, int32_t st_acc, uint32_t st_tot,
                                                 const int32_t *p_acc, const uint32_t *p_tot, int32_t *ranks)
{
    BodyRegs r{0, 0, 0u, 0u};
    const int g1 = g0 + kb;
    for (int j0 = g0; j0 < g1; j0 += 4) {   // four steps per turn, so that their LDS reads overlap
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int j = j0 + u < g1 ? j0 + u : g1 - 1;
            const bool in = j0 + u < g1;
            const int32_t aj = p_acc[j];
            const uint32_t tj = p_tot[j];
            r.pa += (int32_t)(in & ((aj > st_acc) | ((aj == st_acc) & (j < lane))));   // (no short-circuit: no branches)
            r.ps += (int32_t)(in & ((tj < st_tot) | ((tj == st_tot) & (j < lane))));
        }
    }
    wave_sync();   // (an earlier body's ranks have been read)
    ranks[lane] = r.pa;
    ranks[64 + lane] = r.ps;
    wave_sync();
    for (int j0 = g0; j0 < g1; j0 += 4) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int j = j0 + u < g1 ? j0 + u : g1 - 1;
            const uint32_t bit = j0 + u < g1 ? 1u << (j - g0) : 0u;
            r.ma |= ranks[j] < lane ? bit : 0u;
            r.ms |= ranks[64 + j] < lane ? bit : 0u;
        }
    }
    return r;
}
__device__ __forceinline__ void body_store(uint8_t *body, int g0, int kb, int lane, int32_t st_acc,
                                           uint32_t st_tot, int32_t acc_base, const BodyRegs &r)
{
    const uint32_t re = body_re((uint32_t)kb);
    uint16_t *k_acc = (uint16_t *)body;
    uint32_t *k_tot = (uint32_t *)(body + 2 * re);
    uint32_t *m_a = (uint32_t *)(body + 6 * re);
    uint32_t *m_s = (uint32_t *)(body + 10 * re);
    if (lane >= g0 && lane < g0 + kb) {
        k_acc[r.pa] = (uint16_t)(st_acc - acc_base + 1);
        k_tot[r.ps] = st_tot;
    }
    if (lane >= kb && lane < (int)re) {  // sentinels behind the keys (any lane will do)
        k_acc[lane] = 0;
        k_tot[lane] = 0xFFFFFFFFu;
    }
    if (lane < (int)re) { m_a[lane] = r.ma; m_s[lane] = r.ms; }   // lanes beyond kb hold the full set
}

// Whether a step's latency would read as what follows its line (lane j < K holding step j).
__device__ __forceinline__ bool line_ends_odd(int lane, int32_t K, uint32_t st_tot)
{
    return __ballot((lane == 15 || lane == 46) && lane < K && st_tot >= kLineMaxTot) != 0ull;
}
// The lines of slice s (internal.h) by one wavefront, lane j < K holding step j and its caller row.  usable: the slice's accuracies fit
// the keys (and, where entries name steps instead of rows, it has a header that leads to them); `trunc`: it has more steps.
__device__ __forceinline__ void store_lines(const IndexView &ix, int32_t S, int32_t s, int32_t K, bool usable, bool trunc, int lane, int32_t st_acc, uint32_t st_tot,
                                            int32_t row, int32_t acc_base)
{
    const uint32_t n = usable ? (uint32_t)K : 0u;
    const uint32_t lo = ((uint32_t)(st_acc - acc_base + 1) << ix.line_shift()) | (ix.line_rows() ? (uint32_t)row : (uint32_t)lane);
    // lane j's place among the entries: steps 0-15, 16-30, 31-46, 47-61
    const uint32_t j = (uint32_t)lane, plane = (uint32_t)(j >= 16u) + (uint32_t)(j >= 31u) + (uint32_t)(j >= 47u), i = j - line_step0(plane);
    uint2 *line = (uint2 *)(ix.lines + plane * line_plane(S) + (uint32_t)s * kLineBytes);
    // (a plane that the slice does not get to is not read and not written; lane 62 has no step, and writes the last entry of plane 3)
    const bool reached = plane == 0u || (plane == 1u ? n >= 16u : plane == 2u ? n > 31u : n >= 47u);
    const bool is_step = j < n;
    const uint32_t end = usable ? (trunc ? kLineRank : kLineEnd) : kLineRank;
    uint32_t what = kLineEnd;
    if (j == 15u && !usable) what = kLineRank;   // nothing of the slice is in its lines
    if (j == 62u) what = end;
    if (reached && j < 63u) line[line_place(i)] = is_step ? make_uint2(lo, st_tot) : make_uint2(0u, what);
    if (lane == 63 && n >= 16u)   // plane 1 has 15 steps: its last entry tells whether there are more
        ((uint2 *)(ix.lines + line_plane(S) + (uint32_t)s * kLineBytes))[line_place(15u)] = make_uint2(0u, n > 31u ? kLineMore : kLineEnd);
}

constexpr int kBuildWaves = 4;                    // slices (wavefronts) per workgroup

// Highest accuracy and lowest latency-plus-queue over entries [lo, hi) of a slice (hi - lo > 0; lo a multiple
// of 4), for every lane of the wavefront.
__device__ __forceinline__ void range_extremes(const int32_t *acc, const uint32_t *tot, int32_t lo, int32_t hi, int lane,
                                               int32_t &mx, uint32_t &mn)
{
    mx = INT32_MIN;
    mn = 0xFFFFFFFFu;
    for (int32_t i0 = lo; i0 < hi; i0 += 1024) {   // (the entries that pad a slice to a multiple of 4 change nothing)
        v4i a[4];
        uint4 t[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {   // (past the end: the first entries again)
            const int32_t i = i0 + 256 * k + 4 * lane;
            a[k] = *(const v4i *)(acc + (i < hi ? i : lo));
            t[k] = *(const uint4 *)(tot + (i < hi ? i : lo));
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int32_t a01 = a[k].x > a[k].y ? a[k].x : a[k].y, a23 = a[k].z > a[k].w ? a[k].z : a[k].w, m4 = a01 > a23 ? a01 : a23;
            const uint32_t t01 = t[k].x < t[k].y ? t[k].x : t[k].y, t23 = t[k].z < t[k].w ? t[k].z : t[k].w, n4 = t01 < t23 ? t01 : t23;
            mx = m4 > mx ? m4 : mx;
            mn = n4 < mn ? n4 : mn;
        }
    }
    for (int o = 32; o; o >>= 1) {
        const int32_t om = __shfl_xor(mx, o);
        const uint32_t on = __shfl_xor(mn, o);
        mx = om > mx ? om : mx;
        mn = on < mn ? on : mn;
    }
}
// 256 keys of 32 or 64 bits in ascending order by one wavefront, four per lane (key 4 * lane + j is k[j]): a bitonic sort whose
// exchanges stay inside the vector units but for those 16 and 32 lanes apart.  Of two keys a lane keeps the median of
// them and all zeros (the lower) or all ones (the higher), one instruction for 32 bits.  bit[i]: all ones in the lanes
// that hold keys with bit i + 2 in their number.
template <int kLanes>
__device__ __forceinline__ uint32_t from_lane_xor(uint32_t v)
{
    if constexpr (kLanes == 1) return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xF, 0xF, true);           // quad_perm
    else if constexpr (kLanes == 2) return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x4E, 0xF, 0xF, true);
    else if constexpr (kLanes == 4)                                                     // row_half_mirror (7), quad_perm (3)
        return (uint32_t)__builtin_amdgcn_mov_dpp(__builtin_amdgcn_mov_dpp((int)v, 0x141, 0xF, 0xF, true), 0x1B, 0xF, 0xF, true);
    else if constexpr (kLanes == 8) return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x128, 0xF, 0xF, true);     // row_ror:8
    else if constexpr (kLanes == 16) return (uint32_t)__builtin_amdgcn_ds_swizzle((int)v, 0x401F);
    else return (uint32_t)__shfl_xor((int)v, kLanes);
}
template <int kLanes>
__device__ __forceinline__ unsigned long long from_lane_xor(unsigned long long v)
{
    return ((unsigned long long)from_lane_xor<kLanes>((uint32_t)(v >> 32)) << 32) | from_lane_xor<kLanes>((uint32_t)v);
}
__device__ __forceinline__ uint32_t lower_or_higher(uint32_t x, uint32_t y, uint32_t ones)
{
    const uint32_t lo = x < y ? x : y, hi = x < y ? y : x, m = hi < ones ? hi : ones;
    return lo > m ? lo : m;
}
__device__ __forceinline__ unsigned long long lower_or_higher(unsigned long long x, unsigned long long y, uint32_t ones)
{
    return ((x < y) != (ones != 0u)) ? x : y;
}
constexpr int log2_of(int n) { return n > 1 ? 1 + log2_of(n / 2) : 0; }
template <int kSize, int kStride, class Key>
__device__ __forceinline__ void sort_stages(Key (&k)[4], const uint32_t (&bit)[7])
{
    if constexpr (kStride >= 4) {
        const uint32_t ones = bit[log2_of(kStride) - 2] ^ bit[log2_of(kSize) - 2];
#pragma unroll
        for (int j = 0; j < 4; ++j) k[j] = lower_or_higher(k[j], from_lane_xor<kStride / 4>(k[j]), ones);
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (j & kStride) continue;
            const uint32_t ones = kSize >= 4 ? bit[(kSize >= 4 ? log2_of(kSize) : 2) - 2] : (j & kSize) ? ~0u : 0u;
            const Key x = k[j], y = k[j + kStride];
            k[j] = lower_or_higher(x, y, ones);
            k[j + kStride] = lower_or_higher(x, y, ~ones);
        }
    }
    if constexpr (kStride > 1) sort_stages<kSize, kStride / 2>(k, bit);
    else if constexpr (kSize < 256) sort_stages<kSize * 2, kSize>(k, bit);
}
template <class Key>
__device__ __forceinline__ void sort_keys(Key (&k)[4], int lane)
{
    uint32_t bit[7];
#pragma unroll
    for (int i = 0; i < 7; ++i) bit[i] = ((lane >> i) & 1) ? ~0u : 0u;   // (bit[6]: no lane)
    sort_stages<2, 1>(k, bit);
}
// Inclusive scan over the lanes (row_shr 1, 2, 4, 8, then row_bcast 15 and 31); `none` changes nothing.
template <class T, class Op>
__device__ __forceinline__ T scan_lanes(T v, T none, Op op)
{
    v = op(v, (T)__builtin_amdgcn_update_dpp((int)none, (int)v, 0x111, 0xF, 0xF, false));
    v = op(v, (T)__builtin_amdgcn_update_dpp((int)none, (int)v, 0x112, 0xF, 0xF, false));
    v = op(v, (T)__builtin_amdgcn_update_dpp((int)none, (int)v, 0x114, 0xF, 0xF, false));
    v = op(v, (T)__builtin_amdgcn_update_dpp((int)none, (int)v, 0x118, 0xF, 0xF, false));
    v = op(v, (T)__builtin_amdgcn_update_dpp((int)none, (int)v, 0x142, 0xA, 0xF, false));
    return op(v, (T)__builtin_amdgcn_update_dpp((int)none, (int)v, 0x143, 0xC, 0xF, false));
}
// TableView::rank_nodes (`nodes`: the slice's first) of entries [lo, hi) of a slice of L by one wavefront; lo is
// a multiple of 256, hi too unless it is L; (mx, mn): what entries [0, lo) come to.  Four consecutive
// entries per lane, so that the scan over the lanes is done once per 256 entries.
// Bound by the instructions of the sort, 36 stages in a row, which slices of up to kRankUnsorted entries go without.  Measured
// (us, load report and build, every slice truncated): 1600 slices of 2000 entries 77 with 64-bit keys exchanged through
// LDS, 57 so; 1600 of 500, sorted or not, 47 and 37; 8 of 20,000, where a quarter of a slice is one wavefront's, 102 and 48.
// Without any nodes these builds take 46, 36 and 16; the first selection behind them that finds nodes gets back more.
// kSort false: for kernels of tables without longer ones.
template <bool kSort>
__device__ __forceinline__ void write_rank_nodes(const int32_t *acc, const uint32_t *tot, uint4 *nodes, int32_t L, int32_t lo,
                                                 int32_t hi, int lane, int32_t mx, uint32_t mn, int32_t acc_base)
{
    const auto higher = [](int32_t x, int32_t y) { return x > y ? x : y; };
    const auto lower = [](uint32_t x, uint32_t y) { return x < y ? x : y; };
    uint2 *out = (uint2 *)nodes;   // pairs
    uint4 *sorted = nodes + (int64_t)all_level_nodes(L) * 8;
    if (lo >= hi) return;
    int32_t at_next = lo + 4 * lane < hi ? lo + 4 * lane : lo;
    v4i a_next = *(const v4i *)(acc + at_next);   // (the next chunk's entries are requested a chunk ahead)
    uint4 t_next = *(const uint4 *)(tot + at_next);
    for (int32_t c = lo; c < hi; c += kRankBlock) {
        const int32_t i = c + 4 * lane;
        const bool in = i < hi;
        const v4i a = a_next;
        const uint4 t = t_next;
        at_next = i + kRankBlock < hi ? i + kRankBlock : lo;
        a_next = *(const v4i *)(acc + at_next);
        t_next = *(const uint4 *)(tot + at_next);
        int32_t m = in ? higher(higher(a.x, a.y), higher(a.z, a.w)) : INT32_MIN;
        uint32_t n = in ? lower(lower(t.x, t.y), lower(t.z, t.w)) : 0xFFFFFFFFu;
        m = higher(scan_lanes(m, INT32_MIN, higher), mx);
        n = lower(scan_lanes(n, 0xFFFFFFFFu, lower), mn);
        // level 1: the last lane of every four, where the four begin inside the slice
        if ((lane & 3) == 3 && c + 4 * (lane - 3) < hi) out[(uint32_t)(c >> 4) + (lane >> 2)] = make_uint2((uint32_t)m, n);
        mx = __builtin_amdgcn_readlane(m, 63);
        mn = (uint32_t)__builtin_amdgcn_readlane((int)n, 63);
        if (lane == 0) {   // the levels above, where one of their places ends with this chunk
            uint32_t at = 0;
            for (int level = 2; level_nodes(L, level - 1) > 1; ++level) {
                at += 16u * (uint32_t)level_nodes(L, level - 1);
                const int64_t end = (int64_t)c + kRankBlock, size = (int64_t)1 << (4 * level);
                if ((end & (size - 1)) == 0 || end >= L) out[at + (uint32_t)(c >> (4 * level))] = make_uint2((uint32_t)mx, mn);
            }
        }
        if (!kSort || L <= kRankUnsorted) continue;
        // The block by falling accuracy.  Entries that nothing selects (masked, past the end of the slice) come last, as
        // the lowest accuracy there is; among equal ones any order will do, as the search looks at the last of them.
        int ln = lane;
        asm volatile("" : "+v"(ln));   // (the masks of the sort's stages are made here, every time: before the loop there are too many to keep)
        constexpr uint32_t kDead = 0xFFFFFFu;   // accuracies are counted down from kDead - 1 where they fit 24 bits ...
        const uint32_t below[4] = {(uint32_t)a.x - (uint32_t)acc_base, (uint32_t)a.y - (uint32_t)acc_base,
                                   (uint32_t)a.z - (uint32_t)acc_base, (uint32_t)a.w - (uint32_t)acc_base};
        const uint32_t tt[4] = {in ? t.x : 0xFFFFFFFFu, in ? t.y : 0xFFFFFFFFu, in ? t.z : 0xFFFFFFFFu, in ? t.w : 0xFFFFFFFFu};
        bool wide = false;
#pragma unroll
        for (int j = 0; j < 4; ++j) wide = wide | ((tt[j] != 0xFFFFFFFFu) & (below[j] >= kDead));
        int32_t s_acc[4];
        uint32_t s_tot[4];
        if (__ballot(wide) == 0ull) {
            uint32_t k[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) k[j] = ((tt[j] != 0xFFFFFFFFu ? kDead - 1u - below[j] : kDead) << 8) | (uint32_t)(4 * lane + j);
            sort_keys(k, ln);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const bool dead = (k[j] >> 8) == kDead;
                s_acc[j] = dead ? INT32_MIN : (int32_t)((uint32_t)acc_base + (kDead - 1u - (k[j] >> 8)));
                s_tot[j] = tot[dead ? c : c + (int32_t)(k[j] & 0xFFu)];
                s_tot[j] = dead ? 0xFFFFFFFFu : s_tot[j];
            }
        } else {               // ... and are compared as they are where they do not
            unsigned long long k[4];
            const int32_t av[4] = {a.x, a.y, a.z, a.w};
#pragma unroll
            for (int j = 0; j < 4; ++j) k[j] = tt[j] != 0xFFFFFFFFu ? ((unsigned long long)(~((uint32_t)av[j] ^ 0x80000000u)) << 32) | tt[j] : ~0ull;
            sort_keys(k, ln);
#pragma unroll
            for (int j = 0; j < 4; ++j) { s_acc[j] = (int32_t)(~(uint32_t)(k[j] >> 32) ^ 0x80000000u); s_tot[j] = (uint32_t)k[j]; }
        }
        // each with the lowest latency up to it
#pragma unroll
        for (int j = 1; j < 4; ++j) s_tot[j] = lower(s_tot[j], s_tot[j - 1]);
        const uint32_t upto = scan_lanes(s_tot[3], 0xFFFFFFFFu, lower);
        uint32_t before = (uint32_t)__shfl_up((int)upto, 1);
        before = lane ? before : 0xFFFFFFFFu;
        uint2 pair[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) pair[j] = make_uint2((uint32_t)s_acc[j], lower(s_tot[j], before));
        uint4 *blk = sorted + (int64_t)(c / kRankBlock) * kRankBlockNodes * 8;
        blk[8 + 2 * lane] = make_uint4(pair[0].x, pair[0].y, pair[1].x, pair[1].y);
        blk[8 + 2 * lane + 1] = make_uint4(pair[2].x, pair[2].y, pair[3].x, pair[3].y);
        if ((lane & 3) == 3) ((uint2 *)blk)[lane >> 2] = pair[3];
    }
    if (hi == L && lane < 15) {   // the places past the end of every level
        uint32_t at = 0;
        for (int level = 1;; ++level) {
            const int32_t n = level_nodes(L, level);
            const int64_t place = (((int64_t)L + ((int64_t)1 << (4 * level)) - 1) >> (4 * level)) + lane;
            if (place < (int64_t)n * 16) out[at + (uint32_t)place] = make_uint2(0x7FFFFFFFu, 0u);
            if (n <= 1) break;
            at += 16u * (uint32_t)n;
        }
    }
}
// What write_rank_nodes needs of slice s = (t, b), taken from the kernel's arguments (ta, ia, tb, ib, in this
// order) where it is needed: kept from the start of the kernel, for the few slices that have a use for it, it
// pushes other scalars out of their registers.
struct SliceColumns {
    const int32_t *acc;
    const uint32_t *tot;
    uint4 *nodes;
    int32_t L, acc_base;
};
template <bool kTwo>
__device__ __forceinline__ SliceColumns slice_columns(int32_t s, int32_t t, int32_t b)
{
    static_assert(sizeof(TableView) % alignof(IndexView) == 0 && sizeof(IndexView) % alignof(TableView) == 0, "no gaps between the arguments");
    const __attribute__((address_space(4))) char *args = (const __attribute__((address_space(4))) char *)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(args));   // (reads of the arguments are not moved in front of this)
    if (kTwo && blockIdx.y) args += sizeof(TableView) + sizeof(IndexView);
    const __attribute__((address_space(4))) TableView *tv = (const __attribute__((address_space(4))) TableView *)args;
    const int64_t col = (int64_t)b * tv->Vp + tv->seg_off[t];
    return SliceColumns{tv->acc_r + col, tv->tot_r + col, (uint4 *)((char *)tv->rank_hdr + (rank_nodes_at(tv->S) - rank_hdr_at(tv->S))) + (uint64_t)tv->rank_hdr[s].z * 8, tv->seg_len[t], tv->acc_base};
}

// Worker selection: the workers of the steps, like k_step_workers (worker_kernels.hip) makes them when the workers have changed and the
// index has not.  Behind a state report it is a launch less (reports and 1M queries on 20,000 variants 54.1 us per turn with it, 50.2
// so).  Builds of one table do without: 0.4 us of every load report's build, for handles that mostly have no workers.
__device__ __forceinline__ int32_t worker_of_row(const StepFill &f, int32_t row)
{
    if (f.by_row) return f.by_row[row];
    const int32_t c = f.cls[row];
    return c >= 0 ? f.best[c] : -1;
}
__device__ __forceinline__ void store_step_worker(const IndexView &ix, int32_t s, int step, uint32_t at, int32_t worker)
{
    ix.step_worker[at] = worker;
    if (ix.hot_worker && (uint32_t)step < ix.hot_rows)
        ix.hot_worker[(uint32_t)s * ix.hot_rows + (uint32_t)step] = (uint32_t)worker < 0xFFFFu ? (uint16_t)worker : (uint16_t)0xFFFFu;
}
// Thread `at` of `threads`, with nothing else left to do.
__device__ __forceinline__ void store_row_workers(const TableView &tv, const IndexView &ix, int32_t at, int32_t threads)
{
    if (at == 0) ix.step_worker[0] = -1;
    if (ix.fill.rows)
        for (int32_t v = at; v < tv.V; v += threads) ix.fill.rows[v] = worker_of_row(ix.fill, v);
}

// One wavefront per slice, kBuildWaves slices per workgroup.  An entry of the slice is a step exactly
// when no entry ranked before it has at least its accuracy and at most its latency-plus-queue; that
// relation is transitive, so it is enough to test an entry against the earlier STEPS.  The wavefront
// takes in a chunk of the rank-ordered columns, kBuildPer (4, 8, 16 or 32) entries per lane, in registers.  Then
//   1. (first chunk) the steps among the first 64 entries: the first of them is a step (nothing
//      earlier is left), it retires what it dominates among the 64, the next one left is a step, ...;
//   2. a coarse filter: from the steps known so far, a table over ~32 accuracy buckets of the lowest
//      latency-plus-queue among the steps that are at least as accurate as EVERYTHING in the bucket;
//      an entry at or above its bucket's value is dominated for certain and dropped (one LDS read
//      and a compare per entry; nine entries in ten go here).  The others are compacted into a list
//      of candidates in LDS, in rank order;
//   3. rounds over the list until it is empty: the candidates are tested exactly against the steps
//      they have not been tested against yet (four blocks of 64 at a time, a step's values read
//      from its lane once per group; survivors compacted in place), then the steps among the first
//      64 survivors are found as in 1 and leave the list.
// Steps come out in rank order, so when a slice has more than the index keeps, the ones kept are
// its first ones.  The steps sit one per lane (and in LDS); the same wavefront computes the bodies.
// Room in the pool is taken by ONE 64-bit add per workgroup (with one per slice, every slice waited
// microseconds for its turn at the counter).
// kTwo: workgroups (x, 0) build the index of `ta`, (x, 1) that of `tb` (the two tables of a state-aware handle);
// otherwise there is only `ta`.
template <int kBuildPer, bool kTwo>
__global__ __launch_bounds__(64 * kBuildWaves) void k_index_build(TableView ta, IndexView ia, TableView tb, IndexView ib)
{
    const TableView tv = kTwo && blockIdx.y ? tb : ta;
    const IndexView ix = kTwo && blockIdx.y ? ib : ia;
    constexpr int kBuildChunk = 64 * kBuildPer;   // entries of a slice taken in at a time
    __shared__ int32_t c_acc_all[kBuildWaves][kBuildChunk];    // candidates: accuracy,
    __shared__ uint32_t c_tot_all[kBuildWaves][kBuildChunk];   //   latency + queue,
    __shared__ uint16_t c_pos_all[kBuildWaves][kBuildChunk];   //   position in the chunk
    __shared__ int32_t p_acc_all[kBuildWaves][64];             // steps, in rank order
    __shared__ uint32_t p_tot_all[kBuildWaves][64];
    __shared__ int32_t p_pos_all[kBuildWaves][64];
    __shared__ uint32_t f_tab_all[kBuildWaves][64];            // the coarse filter's table
    __shared__ int32_t ranks_all[kBuildWaves][128];            // scratch of body_compute
    __shared__ uint32_t s_size[kBuildWaves], s_steps[kBuildWaves], s_stat[4];
    __shared__ uint32_t s_group[kBuildWaves], s_off[kBuildWaves], s_rec[kBuildWaves];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int32_t *c_acc = c_acc_all[wave], *p_acc = p_acc_all[wave], *p_pos = p_pos_all[wave];
    uint32_t *c_tot = c_tot_all[wave], *p_tot = p_tot_all[wave], *f_tab = f_tab_all[wave];
    uint16_t *c_pos = c_pos_all[wave];
    const int32_t s = (int32_t)blockIdx.x * kBuildWaves + wave;
    const bool inside = s < tv.S;
    const int32_t t = inside ? s / tv.B : 0, b = inside ? s - t * tv.B : 0;
    const int32_t seg = tv.seg_off[t], L = inside ? tv.seg_len[t] : 0;
    const int32_t *__restrict__ accc = tv.acc_r + (int64_t)b * tv.Vp + seg;
    const uint32_t *__restrict__ totc = tv.tot_r + (int64_t)b * tv.Vp + seg;

    // ---- phase A: the steps, in rank order; lane j < K holds step j, p_acc / p_tot / p_pos all of them
    int32_t K = 0;
    bool trunc = false;
    int32_t st_acc = 0, st_pos = 0;
    uint32_t st_tot = 0u;
    // Steps among up to 64 candidates held one per lane, lanes [0, nh), in rank order, none of them
    // dominated by a known step.  The new steps are appended to the step registers.
    auto take_head = [&](int32_t nh, int32_t a, uint32_t tt, int32_t pos) {
        bool alive = lane < nh;
        uint64_t rest = __ballot(alive);
        while (rest) {   // candidate l is a step (nothing alive precedes it): retire what it dominates
            const int l = __builtin_ctzll(rest);
            const int32_t al = __builtin_amdgcn_readlane(a, l);
            const uint32_t tl = (uint32_t)__builtin_amdgcn_readlane((int)tt, l);
            alive = alive & !((l < lane) & (al >= a) & (tl <= tt));
            rest = __ballot(alive) & ~((2ull << l) - 1ull);
        }
        const uint64_t ok = __ballot(alive);
        const int32_t k_new = (int32_t)__builtin_popcountll(ok);
        const int32_t at = K + (int32_t)lanes_below(ok);
        if (alive && at < kIndexCap) { p_acc[at] = a; p_tot[at] = tt; p_pos[at] = pos; }
        trunc = K + k_new > kIndexCap;   // more steps than the index keeps: its first ones stay
        K = trunc ? kIndexCap : K + k_new;
        wave_sync();
        st_acc = lane < K ? p_acc[lane] : 0;
        st_tot = lane < K ? p_tot[lane] : 0u;
        st_pos = lane < K ? p_pos[lane] : 0;
    };
    for (int32_t c0 = 0; c0 < L && !trunc; c0 += kBuildChunk) {
        const int32_t n = L - c0 < kBuildChunk ? L - c0 : kBuildChunk;
        int32_t va[kBuildPer];
        uint32_t vt[kBuildPer];
        uint32_t dead = 0u;   // bit k: entry k of this lane is outside the chunk, dominated, or taken care of
#pragma unroll
        for (int k = 0; k < kBuildPer; ++k) {   // unconditional loads (clamped), so that they overlap
            const int32_t i = k * 64 + lane;
            const int32_t j = c0 + (i < n ? i : n - 1);
            va[k] = accc[j];
            vt[k] = totc[j];
            dead |= i >= n ? 1u << k : 0u;
        }
        if (K == 0) {   // 1. nothing is known yet: the first 64 entries, exactly
            take_head(n < 64 ? n : 64, va[0], vt[0], c0 + lane);
            if (trunc) break;
            dead |= 1u;
        }
        // 2. coarse filter.  Accuracies from the lowest (mn) to the highest (mx) of the steps are cut
        // into buckets of 2^sh; table entry 0 is for entries below mn, entry 1 + q for bucket q, entry
        // 33 for entries above mx.
        {
            int32_t mn = p_acc[0], mx = mn;
            for (int j0 = 1; j0 < K; j0 += 8) {   // (eight per turn: the LDS reads overlap)
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int32_t aj = p_acc[j0 + u < K ? j0 + u : 0];
                    mn = aj < mn ? aj : mn;
                    mx = aj > mx ? aj : mx;
                }
            }
            const uint32_t range = (uint32_t)mx - (uint32_t)mn;
            const int bits = 32 - __builtin_clz(range | 1u);
            const uint32_t sh = bits > 5 ? (uint32_t)(bits - 5) : 0u;   // range >> sh < 32
            // lane i: the lowest latency-plus-queue among the steps at least as accurate as all of
            // bucket i, i.e. with (accuracy - mn + 1) >> sh >= i (entry 0: every step); none: all ones
            uint32_t f = 0xFFFFFFFFu;
            for (int j0 = 0; j0 < K; j0 += 4) {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int j = j0 + u < K ? j0 + u : 0;   // (step 0 again: harmless)
                    const uint64_t uj = (uint64_t)((uint32_t)p_acc[j] - (uint32_t)mn) + 1u;
                    const uint32_t tj = p_tot[j];
                    const bool covers = (uint32_t)(uj >> sh) >= (uint32_t)lane;
                    f = (covers & (tj < f)) ? tj : f;
                }
            }
            f_tab[lane] = lane <= 33 ? f : 0xFFFFFFFFu;
            if (lane == 33) f_tab[33] = 0xFFFFFFFFu;   // above every step: never dominated
            wave_sync();
#pragma unroll
            for (int k = 0; k < kBuildPer; ++k) {
                const uint32_t u = (uint32_t)va[k] - (uint32_t)mn;
                uint32_t idx = 1u + (u >> sh);
                idx = idx > 33u ? 33u : idx;
                idx = va[k] < mn ? 0u : idx;
                const uint32_t fv = f_tab[idx];
                dead |= ((fv != 0xFFFFFFFFu) & (fv <= vt[k])) ? 1u << k : 0u;
            }
        }
        // what is left becomes the candidate list, entries [beg, end) of the LDS arrays
        int32_t beg = 0, end = 0;
#pragma unroll
        for (int k = 0; k < kBuildPer; ++k) {
            const bool live = !((dead >> k) & 1u);
            const uint64_t m = __ballot(live);
            const int32_t at = end + (int32_t)lanes_below(m);
            if (live) { c_acc[at] = va[k]; c_tot[at] = vt[k]; c_pos[at] = (uint16_t)(k * 64 + lane); }
            end += (int32_t)__builtin_popcountll(m);
        }
        wave_sync();
        // 3. rounds
        int32_t applied = 0;   // the list has been tested exactly against steps [0, applied)
        while (beg < end) {
            // the candidates against the steps they have not met; survivors compacted in place (four
            // blocks are read before anything is written, and written at or below where they were read)
            int32_t out = beg;
            for (int32_t i0 = beg; i0 < end; i0 += 256) {
                int32_t ca[4];
                uint32_t ct[4];
                uint16_t cp[4];
                bool gone[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int32_t i = i0 + u * 64 + lane;
                    const int32_t ci = i < end ? i : beg;
                    ca[u] = c_acc[ci]; ct[u] = c_tot[ci]; cp[u] = c_pos[ci];
                    gone[u] = i >= end;
                }
                for (int j = applied; j < K; ++j) {
                    const int32_t aj = __builtin_amdgcn_readlane(st_acc, j);
                    const uint32_t tj = (uint32_t)__builtin_amdgcn_readlane((int)st_tot, j);
#pragma unroll
                    for (int u = 0; u < 4; ++u) gone[u] = gone[u] | ((aj >= ca[u]) & (tj <= ct[u]));
                }
                wave_sync();
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const uint64_t m = __ballot(!gone[u]);
                    if (!gone[u]) {
                        const int32_t to = out + (int32_t)lanes_below(m);
                        c_acc[to] = ca[u]; c_tot[to] = ct[u]; c_pos[to] = cp[u];
                    }
                    out += (int32_t)__builtin_popcountll(m);
                }
            }
            end = out;
            applied = K;
            wave_sync();
            if (beg >= end) break;
            // the steps among the first 64 of them
            const int32_t nh = end - beg < 64 ? end - beg : 64;
            const int32_t hi = beg + (lane < nh ? lane : 0);
            take_head(nh, c_acc[hi], c_tot[hi], c0 + (int32_t)c_pos[hi]);
            if (trunc) break;
            beg += nh;
        }
    }

    // ---- phase B: one or two bodies of sorted keys and bit sets, computed while the workgroup's
    // request for room in the pool is under way
    const int k0 = K < kBodySteps ? K : kBodySteps, k1 = K - k0;
    const uint32_t r0 = (uint32_t)k0 < ix.hot_rows ? (uint32_t)k0 : ix.hot_rows;
    const uint32_t re0 = body_re(k0), re1 = k1 ? body_re(k1) : 0u;
    const uint32_t rows = (2u * r0 + 3u) & ~3u, size0 = body_bytes(re0);
    const uint32_t size = L > 0 ? rows + size0 + body_bytes(re1) : 0u;   // (a multiple of 4)
    if (lane == 0) {
        s_size[wave] = size; s_steps[wave] = (uint32_t)K;
        s_group[wave] = ix.num_groups > 1 ? (uint32_t)ix.task_group[t] : 0u;
    }
    if (threadIdx.x < 4) s_stat[threadIdx.x] = 0u;
    // caller rows of the steps (requested here, used after the bodies have been computed)
    const int32_t row = lane < K ? tv.orig_r[(int64_t)b * tv.Vp + seg + st_pos] : 0;
    __syncthreads();
    if (threadIdx.x == 0) {
        // room in the pool and in step_row for the slices of the workgroup: one 64-bit add on a pair
        // of counters (bytes in the low word) for every run of slices of one group -- one in all,
        // unless the workgroup straddles two groups.  A slice that its group's region has no room for
        // takes its room behind the regions.
        unsigned long long *whole = (unsigned long long *)(ix.ctrl + kCtlPool);
        for (int w0 = 0; w0 < kBuildWaves;) {
            int w1 = w0;
            uint32_t bytes = 0, steps = 0;
            while (w1 < kBuildWaves && s_group[w1] == s_group[w0]) { bytes += s_size[w1]; steps += s_steps[w1]; ++w1; }
            if (bytes) {
                const uint32_t g = s_group[w0];
                const bool grouped = ix.num_groups > 1;
                unsigned long long *pair = grouped ? (unsigned long long *)(ix.gctrl + 2 * g) : whole;
                const unsigned long long old = atomicAdd(pair, ((unsigned long long)steps << 32) | bytes);
                uint32_t off = (uint32_t)old, rec = (uint32_t)(old >> 32);
                for (int w = w0; w < w1; ++w) {
                    if (!grouped) { s_off[w] = off; s_rec[w] = rec; }
                    else if (off + s_size[w] <= ix.region_bytes && rec + s_steps[w] <= ix.group_step_cap) {
                        s_off[w] = g * ix.region_bytes + off; s_rec[w] = g * ix.group_step_cap + rec;
                    } else if (s_size[w]) {
                        const unsigned long long o2 = atomicAdd(whole, ((unsigned long long)s_steps[w] << 32) | s_size[w]);
                        s_off[w] = (uint32_t)o2; s_rec[w] = (uint32_t)(o2 >> 32);
                    }
                    off += s_size[w]; rec += s_steps[w];
                }
            }
            w0 = w1;
        }
    }
    int32_t hi = st_acc, lo = st_acc;   // (of lane 0, a step whenever the slice has variants)
    hi = __builtin_amdgcn_readfirstlane(hi); lo = hi;
    for (int32_t j0 = 1; j0 < K; j0 += 8) {
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int32_t aj = p_acc[j0 + u < K ? j0 + u : 0];
            hi = aj > hi ? aj : hi;
            lo = aj < lo ? aj : lo;
        }
    }
    const BodyRegs b0 = body_compute(0, k0, lane, st_acc, st_tot, p_acc, p_tot, ranks_all[wave]);
    BodyRegs b1{0, 0, 0u, 0u};
    if (k1) b1 = body_compute(k0, k1, lane, st_acc, st_tot, p_acc, p_tot, ranks_all[wave]);
    // of the first steps' rows the low 16 bits go in front of the body, the bits above into the header
    uint32_t row_hi = 0;
    for (uint32_t j = 0; j < r0; ++j)
        row_hi |= ((uint32_t)__builtin_amdgcn_readlane(row, (int)j) >> 16) << (j * ix.row_hi_bits);
    const bool fill = kTwo && (ix.fill.by_row || ix.fill.cls);
    int32_t worker = -1;
    if (fill && lane < K) worker = worker_of_row(ix.fill, row);
    const bool has = inside && L > 0;
    const bool narrow = (int64_t)hi - (int64_t)tv.acc_base <= 65533 && lo >= tv.acc_base && !line_ends_odd(lane, K, st_tot);   // 16-bit accuracy keys
    // the lines, while the room is waited for (which they depend on only where their entries name steps)
    if (inside && ix.line_rows()) store_lines(ix, tv.S, s, K, !has || narrow, trunc, lane, st_acc, st_tot, row, tv.acc_base);
    __syncthreads();
    const uint32_t off = s_off[wave], rec = s_rec[wave];
    const bool fits = has && (uint64_t)off + size <= ix.pool_bytes && (uint64_t)rec + K <= ix.step_cap &&
                      narrow;
    if (fits) {
        uint8_t *body0 = ix.pool + off + rows;
        body_store(body0, 0, k0, lane, st_acc, st_tot, tv.acc_base, b0);
        if (k1) body_store(body0 + size0, k0, k1, lane, st_acc, st_tot, tv.acc_base, b1);
        if (lane < K) {
            ix.step_row[rec + lane] = row;
            if ((uint32_t)lane < r0)   // in reverse in front of the body
                *(uint16_t *)(body0 - 2 - 2 * lane) = (uint16_t)row;
            if (fill) store_step_worker(ix, s, lane, rec + (uint32_t)lane, worker);
        }
    }
    if (inside && !ix.line_rows()) store_lines(ix, tv.S, s, K, !has || fits, trunc, lane, st_acc, st_tot, row, tv.acc_base);
    if (__builtin_expect(has && (trunc || !fits), 0)) {   // (the wavefront) queries of this slice may go through its entries in rank order
        const SliceColumns sc = slice_columns<kTwo>(s, t, b);
        write_rank_nodes<(64 * kBuildPer > kRankUnsorted)>(sc.acc, sc.tot, sc.nodes, sc.L, 0, sc.L, lane, INT32_MIN, 0xFFFFFFFFu, sc.acc_base);
    }
    if (lane == 0 && inside) {
        // This build places by arrival and reads nobody's entry.  It takes its own out all the same: the build numbers
        // come round, and one of k_index_build_shared must not take an entry of that age for its own.  (The current
        // number instead costs a read of a line that the allocation's atomics keep busy: 42 us instead of 34 for two
        // tables of 1600 slices.)
        ix.slice_room[s] = kRoomNone;
        ((uint32_t *)(tv.rank_hdr + s))[3] = (uint32_t)(has && (trunc || !fits));
        if (fits) {
            const uint32_t y = (re0 << kHdrK0Shift) | (re1 << kHdrK1Shift) | (trunc ? kHdrTrunc : 0u) |
                               ((k1 || trunc) ? kHdrDeep : 0u) | row_hi;
            ix.hdr[s] = make_uint4(off + rows - 4u, y, rec, off + size);
        } else if (has) {   // no body: every query of this slice goes to the rank-ordered scan
            ix.hdr[s] = make_uint4(0u, kEmptyHdrY | kHdrPark | kHdrTrunc | kHdrDeep, 0u, 0u);
        } else {            // no variants: the empty dummy body at offset 0 answers "nothing feasible"
            ix.hdr[s] = make_uint4(0u, kEmptyHdrY, 0u, 4u + body_bytes(2));
        }
        // statistics, gathered per workgroup first: thousands of slices adding to one word of global
        // memory take their turns at ~10 ns each, and the kernel does not end before the last one
        if (fits) {
            atomicMax(&s_stat[0], (uint32_t)k0);
            atomicMax(&s_stat[1], (uint32_t)K);
            if (trunc) atomicAdd(&s_stat[2], 1u);
        } else if (has) {
            atomicAdd(&s_stat[3], 1u);
        }
    }
    __syncthreads();
    if (threadIdx.x < 4 && s_stat[threadIdx.x]) {
        constexpr int word[4] = {kCtlMaxK0, kCtlMaxK, kCtlTrunc, kCtlNoBody};
        const uint32_t v = s_stat[threadIdx.x];
        uint32_t *g = &ix.ctrl[word[threadIdx.x]];
        if (threadIdx.x >= 2) atomicAdd(g, v);
        else if (v > __hip_atomic_load(g, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(g, v);   // (mostly not)
    }
    if (fill) store_row_workers(tv, ix, (int32_t)(blockIdx.x * blockDim.x + threadIdx.x), (int32_t)(gridDim.x * blockDim.x));
}

// Few slices, one per workgroup: the time is one slice's chain of dependent steps, so its four wavefronts take
// every stage together and meet at barriers that order LDS traffic only.  Entries come in chunks of 256 kPer, a
// quarter to each wavefront, kPer per lane in registers.  Then
//   1. (first chunk) the steps among the first 64 entries, every pair of them tested, a quarter of the pairs by
//      each wavefront;
//   2. the coarse filter of k_index_build, its table from a quarter of the steps per wavefront; what passes is
//      compacted into the candidate list, in rank order;
//   3. the list in batches of 256: every candidate against the steps known so far and against every candidate
//      before it in the batch (that a non-step dominates it is enough: whatever dominates that one is a
//      step), a quarter of the tests by each wavefront; the survivors are the batch's steps.
// The four then share the bodies: each counts and collects over a quarter of the steps, the parts are put
// together through LDS, while one of them asks for the room in the pool.
// Bound by latency: a few hundred dependent LDS reads and compares on a lone wavefront per SIMD.  Measured (us,
// config 2's 400 slices of 2000 entries): 21.0 with one wavefront looking for the steps round by round, 15.9 so.
template <int kPer, bool kTwo>
__global__ __launch_bounds__(64 * kBuildWaves) void k_index_build_shared(TableView ta, IndexView ia, TableView tb, IndexView ib)
{
    const TableView tv = kTwo && blockIdx.y ? tb : ta;
    const IndexView ix = kTwo && blockIdx.y ? ib : ia;
    constexpr int kChunk = 64 * kBuildWaves * kPer;       // entries of a slice taken in at a time
    constexpr int kBatch = 256;
    __shared__ int2 c_pair[kChunk < 64 ? 64 : kChunk];    // candidates: accuracy, latency + queue
    __shared__ uint16_t c_pos[kChunk];                    //   position in the chunk
    __shared__ int32_t p_acc[64], p_pos[64];              // steps, in rank order
    __shared__ uint32_t p_tot[64];
    __shared__ uint32_t f_part[kBuildWaves][64], f_tab[kBuildWaves][64];   // the coarse filter's table (one copy per wavefront)
    __shared__ unsigned long long s_alive[kBuildWaves][kBatch / 64];
    __shared__ int32_t s_cnt[kBuildWaves];
    __shared__ int32_t ranks[128];                        // the steps' places in their bodies
    __shared__ uint32_t parts[kBuildWaves][4][64];        // what each wavefront found over its quarter of the steps
    __shared__ uint32_t s_off[1], s_rec[1];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int32_t s = (int32_t)blockIdx.x;
    const int32_t t = s / tv.B, b = s - t * tv.B;
    const int32_t seg = tv.seg_off[t], L = tv.seg_len[t];
    const int32_t *__restrict__ accc = tv.acc_r + (int64_t)b * tv.Vp + seg;
    const uint32_t *__restrict__ totc = tv.tot_r + (int64_t)b * tv.Vp + seg;

    // ---- phase A: the steps, in rank order; p_acc / p_tot / p_pos hold all of them
    int32_t K = 0;
    bool trunc = false;
    // After a barrier: which of the 64 candidates of block u every wavefront has found alive.
    auto survivors = [&](int u) { return s_alive[0][u] & s_alive[1][u] & s_alive[2][u] & s_alive[3][u]; };
    auto grow = [&](int32_t k_new) {   // more steps than the index keeps: its first ones stay
        trunc = K + k_new > kIndexCap;
        K = trunc ? kIndexCap : K + k_new;
    };
    for (int32_t c0 = 0; c0 < L && !trunc; c0 += kChunk) {
        const int32_t n = L - c0 < kChunk ? L - c0 : kChunk;
        int ln = lane;
        asm volatile("" : "+v"(ln));   // (masks made from it stay where they are needed: in front of the loop there are too many to keep)
        int32_t va[kPer];
        uint32_t vt[kPer];
        uint32_t dead = 0u;   // bit k: entry k of this lane is outside the chunk, dominated, or taken care of
#pragma unroll
        for (int k = 0; k < kPer; ++k) {   // unconditional loads (clamped), so that they overlap
            const int32_t i = (wave * kPer + k) * 64 + lane;
            const int32_t j = c0 + (i < n ? i : n - 1);
            va[k] = accc[j];
            vt[k] = totc[j];
            dead |= i >= n ? 1u << k : 0u;
        }
        if (c0 == 0) {   // 1. the first 64 entries
            if (wave == 0) c_pair[lane] = make_int2(va[0], (int32_t)vt[0]);
            lds_barrier();
            const int2 me = c_pair[lane];
            bool gone = lane >= n;
#pragma unroll
            for (int x = 0; x < 64 / kBuildWaves; ++x) {
                const int j = wave * (64 / kBuildWaves) + x;
                const int2 o = c_pair[j];
                gone = gone | ((j < ln) & (o.x >= me.x) & ((uint32_t)o.y <= (uint32_t)me.y));
            }
            const uint64_t m = __ballot(!gone);
            if (lane == 0) s_alive[wave][0] = m;
            lds_barrier();
            const uint64_t ok = survivors(0);
            const int32_t at = (int32_t)lanes_below(ok);
            if (wave == 0 && ((ok >> lane) & 1u) && at < kIndexCap) { p_acc[at] = me.x; p_tot[at] = (uint32_t)me.y; p_pos[at] = lane; }
            if (wave == 0) dead |= 1u;
            grow((int32_t)__builtin_popcountll(ok));
            lds_barrier();
            if (trunc) break;
        }
        int32_t vp[kPer];   // where in the chunk
#pragma unroll
        for (int k = 0; k < kPer; ++k) vp[k] = (wave * kPer + k) * 64 + lane;
        for (int round = 0;; ++round) {
            // 2. coarse filter (see k_index_build): accuracies from the lowest (mn) to the highest (mx) of the steps
            // in buckets of 2^sh; entry 0 is for entries below mn, entry 1 + q for bucket q, entry 33 for those above mx
            {
                int32_t mn = p_acc[lane < K ? lane : 0], mx = mn;
                for (int o = 32; o; o >>= 1) {
                    const int32_t x = __shfl_xor(mn, o), y = __shfl_xor(mx, o);
                    mn = x < mn ? x : mn;
                    mx = y > mx ? y : mx;
                }
                const uint32_t range = (uint32_t)mx - (uint32_t)mn;
                const int bits = 32 - __builtin_clz(range | 1u);
                const uint32_t sh = bits > 5 ? (uint32_t)(bits - 5) : 0u;   // range >> sh < 32
                uint32_t f = 0xFFFFFFFFu;
                for (int j0 = wave; j0 < K; j0 += 4 * kBuildWaves) {
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const int j = j0 + kBuildWaves * u < K ? j0 + kBuildWaves * u : 0;   // (step 0 again: harmless)
                        const uint64_t uj = (uint64_t)((uint32_t)p_acc[j] - (uint32_t)mn) + 1u;
                        const uint32_t tj = p_tot[j];
                        const bool covers = (uint32_t)(uj >> sh) >= (uint32_t)lane;
                        f = (covers & (tj < f)) ? tj : f;
                    }
                }
                f_part[wave][lane] = f;
                lds_barrier();
                uint32_t g = f_part[0][lane];
#pragma unroll
                for (int w = 1; w < kBuildWaves; ++w) g = f_part[w][lane] < g ? f_part[w][lane] : g;
                f_tab[wave][lane] = lane <= 32 ? g : 0xFFFFFFFFu;   // (entry 33, above every step: never dominated)
                wave_sync();
#pragma unroll
                for (int k = 0; k < kPer; ++k) {
                    const uint32_t u = (uint32_t)va[k] - (uint32_t)mn;
                    uint32_t idx = 1u + (u >> sh);
                    idx = idx > 33u ? 33u : idx;
                    idx = va[k] < mn ? 0u : idx;
                    const uint32_t fv = f_tab[wave][idx];
                    dead |= ((fv != 0xFFFFFFFFu) & (fv <= vt[k])) ? 1u << k : 0u;
                }
            }
            // what is left becomes the candidate list
            int32_t mine = 0;
#pragma unroll
            for (int k = 0; k < kPer; ++k) mine += (int32_t)__builtin_popcountll(__ballot(!((dead >> k) & 1u)));
            if (lane == 0) s_cnt[wave] = mine;
            lds_barrier();
            int32_t at = 0, num = 0;
#pragma unroll
            for (int w = 0; w < kBuildWaves; ++w) { at += w < wave ? s_cnt[w] : 0; num += s_cnt[w]; }
#pragma unroll
            for (int k = 0; k < kPer; ++k) {
                const bool live = !((dead >> k) & 1u);
                const uint64_t m = __ballot(live);
                const int32_t to = at + (int32_t)lanes_below(m);
                if (live) { c_pair[to] = make_int2(va[k], (int32_t)vt[k]); c_pos[to] = (uint16_t)vp[k]; }
                at += (int32_t)__builtin_popcountll(m);
            }
            lds_barrier();
            if (num == 0) break;
            // 3. a batch from the front of the list: all of it if there is not much, else so few that the filter,
            // made anew from the steps found, takes most of the rest
            const int32_t m = num <= 160 ? num : round == 0 ? 64 : num < kBatch ? num : kBatch;
            const int blocks = (m + 63) >> 6;
            auto test = [&](auto count) __attribute__((always_inline)) {
                constexpr int kU = decltype(count)::value;   // blocks of 64 candidates
                int2 me[kU];
                bool gone[kU];
#pragma unroll
                for (int u = 0; u < kU; ++u) {
                    gone[u] = u * 64 + lane >= m;
                    me[u] = c_pair[(gone[u] ? 0 : u * 64 + lane)];
                }
                for (int j0 = wave; j0 < K; j0 += 4 * kBuildWaves) {
#pragma unroll
                    for (int x = 0; x < 4; ++x) {
                        const int j = j0 + kBuildWaves * x < K ? j0 + kBuildWaves * x : 0;   // (step 0 again: harmless)
                        const int32_t aj = p_acc[j];
                        const uint32_t tj = p_tot[j];
#pragma unroll
                        for (int u = 0; u < kU; ++u) gone[u] = gone[u] | ((aj >= me[u].x) & (tj <= (uint32_t)me[u].y));
                    }
                }
                for (int j0 = wave; j0 < m; j0 += 4 * kBuildWaves) {
#pragma unroll
                    for (int x = 0; x < 4; ++x) {
                        const int j = j0 + kBuildWaves * x;   // (at or behind m: in front of no candidate)
                        const int2 o = c_pair[(j < m ? j : 0)];
#pragma unroll
                        for (int u = 0; u < kU; ++u)
                            gone[u] = gone[u] | ((j < u * 64 + ln) & (j < m) & (o.x >= me[u].x) & ((uint32_t)o.y <= (uint32_t)me[u].y));
                    }
                }
#pragma unroll
                for (int u = 0; u < kU; ++u) {
                    const uint64_t alive = __ballot(!gone[u]);
                    if (lane == 0) s_alive[wave][u] = alive;
                }
            };
            if (blocks == 1) test(std::integral_constant<int, 1>{});
            else if (blocks == 2) test(std::integral_constant<int, 2>{});
            else test(std::integral_constant<int, 4>{});
            lds_barrier();
            int32_t to = K, k_new = 0;   // wavefront w appends the survivors of block w
#pragma unroll
            for (int u = 0; u < kBatch / 64; ++u) {
                if (u >= blocks) continue;
                const int32_t c = (int32_t)__builtin_popcountll(survivors(u));
                to += u < wave ? c : 0;
                k_new += c;
            }
            if (wave < blocks) {
                const uint64_t ok = survivors(wave);
                to += (int32_t)lanes_below(ok);
                if (((ok >> lane) & 1u) && to < kIndexCap) {
                    const int2 me = c_pair[wave * 64 + lane];
                    p_acc[to] = me.x; p_tot[to] = (uint32_t)me.y; p_pos[to] = c0 + (int32_t)c_pos[wave * 64 + lane];
                }
            }
            grow(k_new);
            lds_barrier();
            if (trunc || m == num) break;
            // the rest of the list, in rank order: a quarter to each wavefront, as the entries were
            const int32_t rest = num - m, share = (((rest + kBuildWaves - 1) / kBuildWaves) + 63) & ~63;   // (at most 64 kPer)
            dead = 0u;
#pragma unroll
            for (int k = 0; k < kPer; ++k) {
                const int32_t i = wave * share + k * 64 + lane;
                const bool in = k * 64 < share && i < rest;
                const int2 e = c_pair[m + (in ? i : 0)];
                va[k] = e.x; vt[k] = (uint32_t)e.y; vp[k] = (int32_t)c_pos[m + (in ? i : 0)];
                dead |= in ? 0u : 1u << k;
            }
            lds_barrier();
        }
    }

    // ---- phase B: wavefront w counts and collects over steps [w q, w q + q), q = K / 4 rounded up
    const int32_t st_acc = lane < K ? p_acc[lane] : 0, st_pos = lane < K ? p_pos[lane] : 0;
    const uint32_t st_tot = lane < K ? p_tot[lane] : 0u;
    const int k0 = K < kBodySteps ? K : kBodySteps, k1 = K - k0;
    const uint32_t r0 = (uint32_t)k0 < ix.hot_rows ? (uint32_t)k0 : ix.hot_rows;
    const uint32_t re0 = body_re(k0), re1 = k1 ? body_re(k1) : 0u;
    const uint32_t rows = (2u * r0 + 3u) & ~3u, size0 = body_bytes(re0);
    const bool has = L > 0;
    // accuracies that do not fit 16-bit keys: no bodies, and no room asked for
    const bool narrow = __ballot(lane < K && (st_acc < tv.acc_base || (int64_t)st_acc - (int64_t)tv.acc_base > 65533)) == 0ull && !line_ends_odd(lane, K, st_tot);
    const uint32_t size = has && narrow ? rows + size0 + body_bytes(re1) : 0u;   // (a multiple of 4)
    // requested now, used at the end: the caller rows of the steps
    const int32_t row = (!(wave & 1) && lane < K) ? tv.orig_r[(int64_t)b * tv.Vp + seg + st_pos] : 0;
    // Room in the pool and in step_row.  Without groups the slices are placed in the order of their
    // numbers, so that the layout does not depend on which workgroup was quicker: when the bodies
    // outgrow the LDS mirror of the lookup kernel, the slices it leaves out are always those of the
    // last tasks.  Every slice publishes what it needs; the last wavefront adds up what the slices
    // before its own need, once they have all said so (below), and that of the last slice leaves the
    // statistics (as a maximum per slice in one word of global memory, every slice waited for its turn there).
    // With groups: room by one add on the group's counter pair, asked for now by one lane and looked at after the sets.
    const bool grouped = ix.num_groups > 1;
    const unsigned long long add = size ? ((unsigned long long)(uint32_t)K << 32) | size : 0ull;
    const unsigned long long published = add | ((size && trunc) ? 1ull << kRoomTrunc : 0ull);
    const uint32_t epoch = ix.ctrl[kCtlEpoch];
    if (threadIdx.x == 0)
        __hip_atomic_store(ix.slice_room + s, published | ((unsigned long long)epoch << 20), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const bool asks = grouped && threadIdx.x == 192 && size != 0u;
    const uint32_t grp = grouped ? (uint32_t)ix.task_group[t] : 0u;
    unsigned long long *whole = (unsigned long long *)(ix.ctrl + kCtlPool);
    unsigned long long old = 0;
    if (asks) old = atomicAdd((unsigned long long *)(ix.gctrl + 2 * grp), add);
    const int q = (K + kBuildWaves - 1) / kBuildWaves, j_lo = wave * q, j_hi = j_lo + q < K ? j_lo + q : K;
    const bool second = lane >= k0;   // this lane's step belongs to the second body
    // 1. the place of every step among the keys of its body: how many steps of the body come before it
    uint32_t before = 0;              // by accuracy (low half) and by latency-plus-queue (high half)
    for (int j0 = j_lo; j0 < j_hi; j0 += 4) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int j = j0 + u < j_hi ? j0 + u : j_hi - 1;
            const bool in = (j0 + u < j_hi) & ((j >= k0) == second);
            const int32_t aj = p_acc[j];
            const uint32_t tj = p_tot[j];
            before += (uint32_t)(in & ((aj > st_acc) | ((aj == st_acc) & (j < lane))));   // (no short-circuit: no branches)
            before += (uint32_t)(in & ((tj < st_tot) | ((tj == st_tot) & (j < lane)))) << 16;
        }
    }
    parts[wave][0][lane] = before;
    lds_barrier();
    before = parts[0][0][lane] + parts[1][0][lane] + parts[2][0][lane] + parts[3][0][lane];
    const int32_t pa = (int32_t)(before & 0xFFFFu), ps = (int32_t)(before >> 16);
    if (wave == 0) { ranks[lane] = pa; ranks[64 + lane] = ps; }
    lds_barrier();
    // 2. the sets: lane p collects A[p] and S[p] of both bodies
    uint32_t ma0 = 0u, ms0 = 0u, ma1 = 0u, ms1 = 0u;
    for (int j0 = j_lo; j0 < j_hi; j0 += 4) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int j = j0 + u < j_hi ? j0 + u : j_hi - 1;
            const bool in = j0 + u < j_hi, first = j < k0;
            const uint32_t bit = in ? 1u << (first ? j : j - k0) : 0u;
            const bool a_in = ranks[j] < lane, s_in = ranks[64 + j] < lane;
            ma0 |= (first & a_in) ? bit : 0u;
            ms0 |= (first & s_in) ? bit : 0u;
            ma1 |= (!first & a_in) ? bit : 0u;
            ms1 |= (!first & s_in) ? bit : 0u;
        }
    }
    parts[wave][0][lane] = ma0; parts[wave][1][lane] = ms0; parts[wave][2][lane] = ma1; parts[wave][3][lane] = ms1;
    if (asks) {
        uint32_t off = (uint32_t)old, rec = (uint32_t)(old >> 32);
        if (off + size <= ix.region_bytes && rec + (uint32_t)K <= ix.group_step_cap) {
            off += grp * ix.region_bytes; rec += grp * ix.group_step_cap;
        } else {   // the group's region has no room: behind the regions
            const unsigned long long o2 = atomicAdd(whole, add);
            off = (uint32_t)o2; rec = (uint32_t)(o2 >> 32);
        }
        s_off[0] = off; s_rec[0] = rec;
    }
    // wavefront 2 the lines, while wavefront 3 waits for the room (which they depend on only where their entries name steps)
    if (wave == 2 && ix.line_rows()) store_lines(ix, tv.S, s, K, !has || narrow, trunc, lane, st_acc, st_tot, row, tv.acc_base);
    if (wave == 3 && (!grouped || s == tv.S - 1)) {
        // What the slices before this one need, lane by lane (with groups only for the statistics).  An entry counts once it carries this
        // build's number.  The wait is bounded: every slice publishes as soon as it knows its steps,
        // whatever the others do, and workgroups start in the order of their numbers; should the
        // entries still not be there after kRoomPolls rounds, the slice goes without a body and
        // its queries are answered by the scan.
        constexpr int kRoomPolls = 1 << 18, kAtOnce = 8;
        unsigned long long sum = 0;
        int32_t most = 0;   // steps of the slice that has most
        bool got = true;
        int polls = 0;
        for (int32_t first = 0; first < s && got; first += 64 * kAtOnce) {   // (a batch of entries is read until all of it is there)
            unsigned long long part;
            int32_t part_most;
            do {
                part = 0;
                part_most = 0;
                bool ok = true;
#pragma unroll
                for (int u = 0; u < kAtOnce; ++u) {
                    const int32_t i = first + 64 * u + lane;
                    const unsigned long long v = __hip_atomic_load(ix.slice_room + (i < s ? i : 0), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    const int32_t k = i < s ? (int32_t)((uint32_t)(v >> 32) & kRoomSteps) : 0;
                    ok = ok && (i >= s || ((uint32_t)v >> 20) == epoch);
                    part += i < s ? v & 0xFFFFFFFF000FFFFFull : 0ull;
                    part_most = k > part_most ? k : part_most;
                }
                got = __ballot(!ok) == 0ull;
                if (!got) __builtin_amdgcn_s_sleep(2);
            } while (!got && ++polls < kRoomPolls);
            sum += part;
            most = part_most > most ? part_most : most;
        }
        for (int o = 32; o; o >>= 1) sum += __shfl_xor(sum, o);
        if (lane == 0 && !grouped) {
            s_off[0] = got ? ix.ctrl[kCtlPool0] + (uint32_t)sum : 0xFFFFFFFFu;
            s_rec[0] = got ? ix.ctrl[kCtlSteps0] + ((uint32_t)(sum >> 32) & kRoomSteps) : 0xFFFFFFFFu;
        }
        if (s == tv.S - 1) {   // the totals and the statistics
            most = (size && K > most) ? K : most;
            for (int o = 32; o; o >>= 1) {
                const int32_t x = __shfl_xor(most, o);
                most = x > most ? x : most;
            }
            most = got ? most : kIndexCap;   // (should the wait have run out: the most there can be, here and of the steps)
            sum += published;
            if (lane == 0) {
                if (!grouped) {
                    ix.ctrl[kCtlPool] = ix.ctrl[kCtlPool0] + (uint32_t)sum;
                    ix.ctrl[kCtlSteps] = got ? ix.ctrl[kCtlSteps0] + ((uint32_t)(sum >> 32) & kRoomSteps) : ix.step_cap;
                }
                ix.ctrl[kCtlTrunc] = (uint32_t)(sum >> kRoomTrunc);
                ix.ctrl[kCtlMaxK] = (uint32_t)most;
                ix.ctrl[kCtlMaxK0] = (uint32_t)(most < 1 ? 1 : most < kBodySteps ? most : kBodySteps);
            }
        }
    }
    lds_barrier();   // (also: the room is in LDS)
    const uint32_t off = s_off[0], rec = s_rec[0];
    const bool fits = has && (uint64_t)off + size <= ix.pool_bytes && (uint64_t)rec + K <= ix.step_cap && narrow;
    uint8_t *body0 = ix.pool + off + rows;
    if (wave == 2 && !ix.line_rows()) store_lines(ix, tv.S, s, K, !has || fits, trunc, lane, st_acc, st_tot, row, tv.acc_base);
    if (wave <= 1 && fits && (wave == 0 || k1)) {   // wavefront 0 writes the first body, wavefront 1 the second
        const int h = 2 * wave;
        BodyRegs r{pa, ps, parts[0][h][lane] | parts[1][h][lane] | parts[2][h][lane] | parts[3][h][lane],
                   parts[0][h + 1][lane] | parts[1][h + 1][lane] | parts[2][h + 1][lane] | parts[3][h + 1][lane]};
        if (wave == 0) body_store(body0, 0, k0, lane, st_acc, st_tot, tv.acc_base, r);
        else body_store(body0 + size0, k0, k1, lane, st_acc, st_tot, tv.acc_base, r);
    }
    if (__builtin_expect(has && (trunc || !fits), 0)) {   // (the whole workgroup) queries of this slice may go through its entries in rank order
        const SliceColumns sc = slice_columns<kTwo>(s, t, b);
        const int32_t quarter = (((sc.L + kBuildWaves - 1) / kBuildWaves) + 255) & ~255;
        const int32_t from = wave * quarter, to = from + quarter < sc.L ? from + quarter : sc.L;
        int32_t mx = INT32_MIN;
        uint32_t mn = 0xFFFFFFFFu;
        range_extremes(sc.acc, sc.tot, from, to, lane, mx, mn);
        lds_barrier();   // (the parts of the bodies have been read)
        if (lane == 0) { parts[wave][0][0] = (uint32_t)mx; parts[wave][0][1] = mn; }
        lds_barrier();
        mx = INT32_MIN;
        mn = 0xFFFFFFFFu;
        for (int w = 0; w < wave; ++w) {
            mx = (int32_t)parts[w][0][0] > mx ? (int32_t)parts[w][0][0] : mx;
            mn = parts[w][0][1] < mn ? parts[w][0][1] : mn;
        }
        write_rank_nodes<(kChunk > kRankUnsorted)>(sc.acc, sc.tot, sc.nodes, sc.L, from, to, lane, mx, mn, sc.acc_base);
    }
    const bool fill = kTwo && (ix.fill.by_row || ix.fill.cls);
    if (wave != 0) {   // (no barrier follows)
        if (fill) store_row_workers(tv, ix, s * 64 * (kBuildWaves - 1) + (int32_t)threadIdx.x - 64, tv.S * 64 * (kBuildWaves - 1));
        return;
    }
    if (fits && lane < K) {
        if (fill) store_step_worker(ix, s, lane, rec + (uint32_t)lane, worker_of_row(ix.fill, row));
        ix.step_row[rec + lane] = row;
        if ((uint32_t)lane < r0)   // in reverse in front of the body
            *(uint16_t *)(body0 - 2 - 2 * lane) = (uint16_t)row;
    }
    uint32_t row_hi = 0;   // of the first steps' rows the bits above the low 16 go into the header
    for (uint32_t j = 0; j < r0; ++j)
        row_hi |= ((uint32_t)__builtin_amdgcn_readlane(row, (int)j) >> 16) << (j * ix.row_hi_bits);
    if (lane == 0) {
        ((uint32_t *)(tv.rank_hdr + s))[3] = (uint32_t)(has && (trunc || !fits));
        if (fits) {
            const uint32_t y = (re0 << kHdrK0Shift) | (re1 << kHdrK1Shift) | (trunc ? kHdrTrunc : 0u) |
                               ((k1 || trunc) ? kHdrDeep : 0u) | row_hi;
            ix.hdr[s] = make_uint4(off + rows - 4u, y, rec, off + size);
        } else if (has) {   // no body: every query of this slice goes to the rank-ordered scan
            ix.hdr[s] = make_uint4(0u, kEmptyHdrY | kHdrPark | kHdrTrunc | kHdrDeep, 0u, 0u);
        } else {            // no variants: the empty dummy body at offset 0 answers "nothing feasible"
            ix.hdr[s] = make_uint4(0u, kEmptyHdrY, 0u, 4u + body_bytes(2));
        }
    }
    if (lane == 0 && has && !fits) atomicAdd(&ix.ctrl[kCtlNoBody], 1u);
}

// ---------------------------------------------------------------- lookup

// A suggestion and its distance as the 16-byte record the first tier of the complete Case I leaves
// beside every query it lists for the second tier (latency overshoot < 2^33, accuracy shortfall < 2^32).
__device__ __forceinline__ v4i pack_side(int32_t row, const HowFar &h)
{
    return v4i{row, (int32_t)(uint32_t)h.over, (int32_t)(uint32_t)h.shortf,
               h.missed | (int32_t)((h.over >> 32) & 1) << 2 | (int32_t)((h.shortf >> 32) & 1) << 3};
}
__device__ __forceinline__ HowFar unpack_side(const v4i &r)
{
    return HowFar{r.w & 3, (int64_t)(uint32_t)r.y | ((int64_t)((r.w >> 2) & 1) << 32),
                  (int64_t)(uint32_t)r.z | ((int64_t)((r.w >> 3) & 1) << 32)};
}

// kMode 0: selection.  1: selection plus closest-variant suggestion (q.closest).
// 2 and 3: the two tiers of the state-aware selection.  2 is the selection over the first tier's
// table; it also writes q.tier (1 = answered, 0 = not) and lists every valid query it leaves
// unanswered, as a (query, latency bound, accuracy bound, slice) record, in its workgroup's part of
// q.open (q.open_cap records each, as many as the workgroup has queries), the number of records in
// q.open_count[workgroup].  3 takes the records of its workgroup's list instead of the query
// arrays, looks them up in the second tier's table and writes q.out and q.tier (= 2) of those it
// can answer; it must be launched with the same grid as the pass that wrote the lists.
// 4 and 5: as 2 and 3, and the worker that serves each answer goes to q.worker (ix.step_worker for
// answers that are steps of the index, q.row_worker for answers found by the scan).
// 6 and 7: as 2 and 3, and q.closest gets the complete Case I: the selected variant, or for a query
// that neither tier can answer the closest variant of the two tiers (6 writes the first tier's
// suggestion, and how far it is from the requirements, beside every record of its lists (q.open_side);
// 7 compares it with its own).  8 and 9: 6 and 7 with the workers of 4 and 5.
template <int kMode>
__global__ __launch_bounds__(kSelThreads) void k_index_select(TableView tv, IndexView ix, QueryView q,
                                                              int32_t *__restrict__ park_mem, uint32_t lds_cap)
{
    constexpr bool kCase1 = kMode >= 6;
    constexpr bool kClosest = kMode == 1, kFirst = kMode >= 2 && !(kMode & 1);
    constexpr bool kSecond = kMode >= 3 && (kMode & 1);
    constexpr bool kWorker = kMode == 4 || kMode == 5 || kMode == 8 || kMode == 9;
    constexpr bool kSuggest = kClosest || kCase1;   // queries without a feasible variant are parked too, for the suggestion
    extern __shared__ __align__(16) uint32_t lds_w[];  // [16 B control][S + 1 headers][lds_cap bytes of bodies]
    publish_index_stats(tv);

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t nhdr = (uint32_t)tv.S + 1u;
    const uint32_t hdr_bytes = lds_header_bytes(tv.S);
    const uint32_t lds_base = (uint32_t)(uintptr_t)(INFAAS_LDS uint32_t *)lds_w;
    const uint32_t lds_hdr0 = lds_base + kLdsCtrlBytes;
    const uint32_t rebase = lds_hdr0 + hdr_bytes;      // LDS address of pool offset 0
    const bool aligned = ((((uintptr_t)q.task) | ((uintptr_t)q.slo) | ((uintptr_t)q.min_acc) |
                           ((uintptr_t)q.bidx) | ((uintptr_t)q.out) | ((uintptr_t)q.closest) |
                           ((uintptr_t)q.tier) | ((uintptr_t)q.worker)) & 15u) == 0;
    // Work units of one wavefront: 64 lanes x kPerThread consecutive queries.  Unit u belongs to
    // workgroup u mod (number of workgroups): all workgroups move through the query arrays together
    // (measured 5% faster than one contiguous range per workgroup).  Inside a workgroup the
    // wavefronts draw its units from a counter in LDS, because the wavefronts of a SIMD do not
    // advance at the same speed.
    // A lane's queries in a unit: four consecutive ones in every block of 256, so that each 16-byte
    // access of the wavefront covers one contiguous kilobyte.
    constexpr int kUnit = 64 * kPerThread;
    constexpr int kSpan = (kPerThread / 4 - 1) * 256 + 4;           // from a lane's first query to behind its last
    auto qoff = [](int k) -> int32_t { return (k >> 2) * 256 + (k & 3); };   // offset of query k of a lane
    // second tier: the units are blocks of 256 records of the workgroup's own list
    const v4i *open_in = (const v4i *)q.open + (int64_t)blockIdx.x * q.open_cap;
    v4i *open_out = (v4i *)q.open + (int64_t)blockIdx.x * q.open_cap;
    const int32_t open_n = kSecond ? q.open_count[blockIdx.x] : 0;
    if (kSecond && open_n == 0) {   // the whole workgroup: nothing was left open in its share
        if (tid < kLookupStats) ix.stats[blockIdx.x * kLookupStats + tid] = 0u;
        if (blockIdx.x == 0 && tid == 0) ix.stats[-1] = gridDim.x;
        return;
    }
    const int32_t nunits = ((kSecond ? open_n : q.n) + kUnit - 1) / kUnit;
    // Query fields of one unit for this lane (unit < 0: nothing left; the fields then describe a
    // query outside the table).  Second tier: tk holds the slice and bi the query's number (negative: no
    // record).
    struct Fields {
        int32_t unit;   // (first: behind bi, the compiler reads bi[k] and it with one wide load, through memory)
        int32_t tk[kPerThread], sl[kPerThread], am[kPerThread], bi[kPerThread];
    };
    constexpr int32_t kNoRecord = -1;
    auto load_unit = [&](Fields &f, int32_t unit) __attribute__((always_inline)) {
        f.unit = unit;
        const int32_t i0 = unit * kUnit + lane * 4;
        if (unit < 0) {
#pragma unroll
            for (int k = 0; k < kPerThread; ++k) { f.tk[k] = kSecond ? tv.S : -1; f.sl[k] = 0; f.am[k] = 0; f.bi[k] = kSecond ? kNoRecord : 0; }
        } else if (kSecond) {
#pragma unroll
            for (int k = 0; k < kPerThread; ++k) {   // record k of a lane: 64 records behind record k - 1
                const int32_t r = unit * kUnit + k * 64 + lane;
                const v4i e = open_in[r < open_n ? r : 0];
                f.tk[k] = r < open_n ? e.w : tv.S;   // (members in the order of the branch above: the compiler
                f.sl[k] = e.y; f.am[k] = e.z;        // merges the branches' last stores, and through a pointer
                f.bi[k] = r < open_n ? e.x : kNoRecord;   // if they go to different members)
            }
        } else if (aligned && i0 + kSpan <= q.n) {
            // one 32-bit byte offset for all four arrays (n <= 2^28).  Loads and stores are
            // non-temporal: every byte is used once.  (With query arrays that come from HBM, as they
            // do when each call gets a new batch, non-temporal loads were measured 4% faster than
            // ordinary ones and ordinary stores 4% slower; only on arrays that a previous call
            // left in the last-level cache are ordinary loads 1% ahead.)
            const uint32_t off = (uint32_t)i0 * 4u;
#pragma unroll
            for (int h = 0; h < kPerThread / 4; ++h) {
                const v4i a = __builtin_nontemporal_load((const v4i *)((const char *)q.task + off) + 64 * h);
                const v4i b = __builtin_nontemporal_load((const v4i *)((const char *)q.slo + off) + 64 * h);
                const v4i c = __builtin_nontemporal_load((const v4i *)((const char *)q.min_acc + off) + 64 * h);
                const v4i d = __builtin_nontemporal_load((const v4i *)((const char *)q.bidx + off) + 64 * h);
                f.tk[4 * h] = a.x; f.tk[4 * h + 1] = a.y; f.tk[4 * h + 2] = a.z; f.tk[4 * h + 3] = a.w;
                f.sl[4 * h] = b.x; f.sl[4 * h + 1] = b.y; f.sl[4 * h + 2] = b.z; f.sl[4 * h + 3] = b.w;
                f.am[4 * h] = c.x; f.am[4 * h + 1] = c.y; f.am[4 * h + 2] = c.z; f.am[4 * h + 3] = c.w;
                f.bi[4 * h] = d.x; f.bi[4 * h + 1] = d.y; f.bi[4 * h + 2] = d.z; f.bi[4 * h + 3] = d.w;
            }
        } else {
#pragma unroll
            for (int k = 0; k < kPerThread; ++k) {
                const int32_t i = i0 + qoff(k);
                const bool in = i < q.n;
                f.tk[k] = in ? q.task[i] : -1;   // -1: outside the table, answered "nothing feasible"
                f.sl[k] = in ? q.slo[i] : 0;
                f.am[k] = in ? q.min_acc[i] : 0;
                f.bi[k] = in ? q.bidx[i] : 0;
            }
        }
    };

    Fields fa, fb;   // two buffers in rotation: searched now, next
    {
        // Mirror the index: all global loads of a lane (its headers and up to kFillDepth x 16 bytes
        // of bodies) are issued before the first LDS write, so the fill costs about one memory
        // round trip.  The whole LDS capacity is copied, used or not, which keeps the copy
        // independent of any value that would have to be read from memory first.
        // Every workgroup copies the same bytes at the same time; the copy goes in 1 KB chunks, one
        // per wavefront and load, and every wavefront of the device starts at a different chunk, so
        // that the requests spread over all L2 channels.
        constexpr int kFillDepth = 10;
        const uint4 *gp = (const uint4 *)ix.pool;
        uint4 *lp = (uint4 *)(lds_w + ((kLdsCtrlBytes + hdr_bytes) >> 2));
        const uint32_t nvec = (lds_cap < ix.pool_bytes ? lds_cap : ix.pool_bytes) >> 4;
        const uint32_t nchunks = (nvec + 63u) >> 6;
        const uint32_t per_wave = (nchunks + (kSelThreads / 64) - 1) / (kSelThreads / 64);
        const uint32_t start = nchunks ? (blockIdx.x * 11u + (uint32_t)wave * per_wave) % nchunks : 0u;
        uint4 v[kFillDepth];
        uint32_t at[kFillDepth];
        bool ok[kFillDepth];
#pragma unroll
        for (int u = 0; u < kFillDepth; ++u) {
            uint32_t c = start + u;
            c = c >= nchunks ? c - nchunks : c;
            ok[u] = (uint32_t)u < per_wave && (uint32_t)wave * per_wave + u < nchunks && c * 64u + lane < nvec;
            at[u] = ok[u] ? c * 64u + lane : 0u;   // lanes with nothing to copy read vector 0 and drop it
            v[u] = gp[at[u]];                      // unconditional: keeps all loads in flight together
        }
        // headers: rebased onto the LDS copy; slices whose bodies are not resident are parked
        for (uint32_t s = tid; s < nhdr; s += kSelThreads) {
            const uint4 g = ix.hdr[s];
            const bool resident = !(g.y & kHdrPark) && g.w <= lds_cap && g.z < 65536u;
            v2u l;
            l.x = ((resident ? g.x : 0u) + rebase) | (g.y << kLdsAddrBits);   // high row bits above the address
            l.y = resident ? ((g.y & 0xFFFF0000u) | g.z) : (kEmptyHdrY | kHdrPark | kHdrDeep);
            *(v2u *)(lds_w + (kLdsCtrlBytes / 4) + s * (kLdsHdrBytes / 4)) = l;
        }
#pragma unroll
        for (int u = 0; u < kFillDepth; ++u)
            lp[at[u]] = v[u];   // unconditional as well (lanes without work rewrite vector 0 with itself)
        for (uint32_t c0 = kFillDepth; c0 < per_wave; ++c0) {   // only if LDS ever exceeds 160 KB
            uint32_t c = start + c0;
            c = c >= nchunks ? c - nchunks : c;
            const uint32_t i = c * 64u + lane;
            if ((uint32_t)wave * per_wave + c0 < nchunks && i < nvec) lp[i] = gp[i];
        }
    }
    // worker selection: 16-bit workers of the hot steps behind the bodies (lds_cap excludes them)
    const bool hot_w = kWorker && ix.hot_worker != nullptr;
    const uint32_t hotw_base = rebase + lds_cap;
    if (hot_w) {
        const uint32_t nw = (nhdr - 1u) * ix.hot_rows;   // 16-bit entries; the array has 8 more behind them
        const uint32_t *gw = (const uint32_t *)ix.hot_worker;
        uint32_t *lw = lds_w + ((kLdsCtrlBytes + hdr_bytes + lds_cap) >> 2);
        for (uint32_t i = tid; i < (nw + 1u) >> 1; i += kSelThreads) lw[i] = gw[i];
    }
    if (tid < (int)(kLdsCtrlBytes / 4)) lds_w[tid] = 0u;
    __syncthreads();

    const uint32_t row_hi_mask = (1u << ix.row_hi_bits) - 1u;
    const int32_t acc_base_m1 = tv.acc_base - 1;   // acc_base is above INT32_MIN
    const uint32_t max_k = ix.ctrl[kCtlMaxK0];
    const int nit = 32 - __builtin_clz(max_k | 1u);    // <= 5
    const LdsMem lmem{};
    const GlobalMem gmem{ix.pool};
    // Parked queries of this wavefront: (query, latency bound, accuracy bound, slice) records in a
    // queue of its own in global memory, written and read by this wavefront only.
    v4i *wq = (v4i *)park_mem + ((int64_t)blockIdx.x * (kSelThreads / 64) + wave) * kWaveQueue;
    uint32_t cnt = 0;   // records in the queue (wave-uniform)
    // what became of this wavefront's parked queries (wave-uniform; summed per workgroup at the end)
    uint32_t st_parked = 0, st_second = 0, st_global = 0, st_scanned = 0, st_none = 0;

    uint32_t &s_next = lds_w[2];
    auto next_unit = [&]() -> int32_t {
        uint32_t u = 0;
        if (lane == 0) u = atomicAdd(&s_next, 1u);
        u = (uint32_t)__builtin_amdgcn_readfirstlane((int)u);
        const int64_t unit = kSecond ? (int64_t)u : (int64_t)blockIdx.x + (int64_t)u * gridDim.x;
        return unit < nunits ? (int32_t)unit : -1;
    };
    load_unit(fa, next_unit());
    load_unit(fb, next_unit());
    // Software pipeline.  A wavefront waits for memory once per unit, at the top, where it needs the
    // unit's query fields; that wait also covers everything requested before it.  The rows gathered
    // for a unit are therefore consumed, and its results stored, only after the NEXT unit's wait --
    // one full unit of LDS work after they were requested -- so neither the gather nor the store
    // latency is exposed.  Two buffers of query fields alternate: as soon as a unit has been searched
    // its buffer is refilled with the unit after the next, which leaves that request one full stage
    // to arrive.  (A third buffer, requested a stage earlier, was measured 1% slower.)
    int32_t p_lrow[kPerThread], p_grow[kPerThread], p_i0 = -1;
    uint32_t p_base[kPerThread];
    bool p_inl[kPerThread];
    int32_t p_qi[kPerThread];   // second tier only: where each result goes
    int32_t p_wk[kPerThread];   // worker selection only: the worker of each answer, gathered from global memory ...
    int32_t p_wl[kPerThread];   // ... or its 16-bit copy from LDS (-1: not there)
    auto p_worker = [&](int k) -> int32_t { return p_wl[k] >= 0 ? (p_wl[k] == 0xFFFF ? -1 : p_wl[k]) : p_wk[k]; };
    auto p_val = [&](int k) -> int32_t { return p_inl[k] ? (int32_t)((p_base[k] << 16) | (uint32_t)p_lrow[k]) : p_grow[k]; };
    auto store_unit = [&]() {
        if (p_i0 < 0) return;
        if (kSecond) {   // only the answers: the first tier has written "none" for all of the list
#pragma unroll
            for (int k = 0; k < kPerThread; ++k)
                if (p_qi[k] >= 0 && p_val(k) >= 0) {
                    q.out[p_qi[k]] = p_val(k); q.tier[p_qi[k]] = 2;
                    if (kCase1) q.closest[p_qi[k]] = p_val(k);
                    if (kWorker) q.worker[p_qi[k]] = p_worker(k);
                }
        } else if (aligned && p_i0 + kSpan <= q.n) {
#pragma unroll
            for (int h = 0; h < kPerThread / 4; ++h) {
                const v4i r = {p_val(4 * h), p_val(4 * h + 1), p_val(4 * h + 2), p_val(4 * h + 3)};
                __builtin_nontemporal_store(r, (v4i *)((char *)q.out + (uint32_t)p_i0 * 4u) + 64 * h);
                if (kSuggest) __builtin_nontemporal_store(r, (v4i *)((char *)q.closest + (uint32_t)p_i0 * 4u) + 64 * h);
                if (kFirst) {
                    const v4i t4 = {r.x >= 0, r.y >= 0, r.z >= 0, r.w >= 0};
                    __builtin_nontemporal_store(t4, (v4i *)((char *)q.tier + (uint32_t)p_i0 * 4u) + 64 * h);
                }
                if (kWorker) {
                    const v4i w4 = {p_worker(4 * h), p_worker(4 * h + 1), p_worker(4 * h + 2), p_worker(4 * h + 3)};
                    __builtin_nontemporal_store(w4, (v4i *)((char *)q.worker + (uint32_t)p_i0 * 4u) + 64 * h);
                }
            }
        } else {
#pragma unroll
            for (int k = 0; k < kPerThread; ++k)
                if (p_i0 + qoff(k) < q.n) {
                    q.out[p_i0 + qoff(k)] = p_val(k);
                    if (kSuggest) q.closest[p_i0 + qoff(k)] = p_val(k);
                    if (kFirst) q.tier[p_i0 + qoff(k)] = p_val(k) >= 0;
                    if (kWorker) q.worker[p_i0 + qoff(k)] = p_worker(k);
                }
        }
    };
    // One pipeline stage: search the unit in `cur`, then request the unit after the next into it.
    uint32_t &s_open = lds_w[3];   // first tier: records in the workgroup's list so far
    // Room for `count` (wave-uniform, > 0) more records in the workgroup's list: one LDS atomic.
    auto open_room = [&](uint32_t count) -> uint32_t {
        uint32_t at = 0;
        if (lane == 0) at = atomicAdd(&s_open, count);
        return (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
    };
    auto stage = [&](Fields &cur) __attribute__((always_inline)) {
        const int32_t i0 = kSecond ? 0 : cur.unit * kUnit + lane * 4;
        store_unit();                                   // results of the previous unit
        // slice header; queries outside the table use the header of the empty slice (entry S)
        uint32_t body[kPerThread], y[kPerThread], rec[kPerThread], keys[kPerThread], dd[kPerThread],
            lim[kPerThread], m[kPerThread], sl_of[kPerThread], rbase[kPerThread];
#pragma unroll
        for (int k = 0; k < kPerThread; ++k) {
            const uint32_t inside = ((uint32_t)cur.tk[k] < (uint32_t)tv.T) & ((uint32_t)cur.bi[k] < (uint32_t)tv.B);
            const uint32_t ok = inside & (uint32_t)(cur.sl[k] >= 0);   // a negative bound admits nothing
            const uint32_t own = __umul24((uint32_t)cur.tk[k], (uint32_t)tv.B) + (uint32_t)cur.bi[k];
            // (a record of the second tier names its slice; one with a negative bound can only get a suggestion)
            const uint32_t s = kSecond ? ((kCase1 && cur.sl[k] < 0) ? (uint32_t)tv.S : (uint32_t)cur.tk[k])
                                       : (ok ? own : (uint32_t)tv.S);
            // the slice a parked record names
            sl_of[k] = kSecond ? (uint32_t)cur.tk[k] : (kSuggest ? (inside ? own : (uint32_t)tv.S) : s);
            const v2u h = lmem.ld64(lds_hdr0 + s * kLdsHdrBytes);
            body[k] = h.x & ((1u << kLdsAddrBits) - 1u); y[k] = h.y; rec[k] = h.y & 0xFFFFu;
            rbase[k] = h.x >> kLdsAddrBits;
            keys[k] = (y[k] >> kHdrK0Shift) & 0x3Fu;   // Re of the first body
            dd[k] = acc_threshold(cur.am[k], acc_base_m1);
            lim[k] = (uint32_t)cur.sl[k];
        }
        search_bodies<kPerThread>(lmem, nit, body, keys, dd, lim, m);
        bool df[kPerThread];
#pragma unroll
        for (int k = 0; k < kPerThread; ++k) {
            const bool hit = m[k] != 0u;
            const uint32_t step = (uint32_t)__builtin_ctzg(m[k], -1);   // no fitting step: above every count
            // row of the step: from in front of the body (low 16 bits) and the header (the bits above)
            // when it is one of its first hot_rows steps, else from step_row in global memory.  Both
            // reads are issued for every lane (lanes that do not need one read a fixed address) and
            // used after the next wait.  step_row[0] is -1, which is what a lane without a fitting
            // step reads and reports.
            const bool inl = step < ix.hot_rows;
            const uint32_t at = inl ? body[k] - 2u * step : body[k];
            p_lrow[k] = (int32_t)lmem.ld16(at, 2u);
            p_base[k] = (rbase[k] >> ((step * ix.row_hi_bits) & 31u)) & row_hi_mask;
            p_grow[k] = *(const int32_t *)((const char *)ix.step_row + ((hit && !inl) ? (rec[k] + step) * 4u : 0u));
            p_inl[k] = inl;
            // the worker of the step: of a hot step from LDS, else by the same kind of gather as the
            // row (entry 0, for no step, is -1)
            if (kWorker) {
                const bool wl = hot_w && inl;
                p_wk[k] = *(const int32_t *)((const char *)ix.step_worker + ((hit && !wl) ? (rec[k] + step) * 4u : 0u));
                p_wl[k] = -1;
                if (hot_w) {   // every lane reads (lanes without a hot step the first entry) and keeps it only if it is its own
                    const uint32_t slice = kSecond ? (uint32_t)cur.tk[k] : sl_of[k];
                    const uint32_t w16 = lmem.ld16(hotw_base + (wl ? (__umul24(slice, ix.hot_rows) + step) * 2u : 0u), 0u);
                    p_wl[k] = wl ? (int32_t)w16 : -1;
                }
            }
            if (kSecond) p_qi[k] = cur.bi[k];
            // parked: a miss that the second body / the scan may still turn into a hit; in the
            // closest-variant mode also every final miss of a query inside the table
            df[k] = !hit && ((int32_t)y[k] < 0 || (kSuggest && sl_of[k] != (uint32_t)tv.S));
            if (kSuggest && (int32_t)y[k] >= 0) sl_of[k] |= kParkFinal;   // nothing feasible: only the suggestion is open
        }
        p_i0 = i0;
#pragma unroll
        for (int k = 0; k < kPerThread; ++k) {
            const uint64_t mask = __ballot(df[k]);
            if (mask) {   // parked queries are always inside the table
                // (first word: the query; in the last pass of the complete Case I the record's place in the
                // workgroup's list, where the query and the first tier's suggestion are found)
                if (df[k]) wq[cnt + lanes_below(mask)] = v4i{(kCase1 && kSecond) ? cur.unit * kUnit + k * 64 + lane : kSecond ? cur.bi[k] : i0 + qoff(k),
                                                              cur.sl[k], cur.am[k], (int32_t)sl_of[k]};
                cnt += (uint32_t)__builtin_popcountll(mask);
                st_parked += (uint32_t)__builtin_popcountll(mask);
            }
        }
        if (kFirst) {   // valid queries that end here without an answer go to the second tier
            uint64_t om[kPerThread];
            uint32_t total = 0;
#pragma unroll
            for (int k = 0; k < kPerThread; ++k) {
                om[k] = __ballot(m[k] == 0u && !df[k] && (sl_of[k] & ~kParkFinal) != (uint32_t)tv.S);
                total += (uint32_t)__builtin_popcountll(om[k]);
            }
            if (total) {
                uint32_t at = open_room(total);
#pragma unroll
                for (int k = 0; k < kPerThread; ++k) {
                    if ((om[k] >> lane) & 1u)
                        open_out[at + lanes_below(om[k])] = v4i{i0 + qoff(k), cur.sl[k], cur.am[k], (int32_t)sl_of[k]};
                    at += (uint32_t)__builtin_popcountll(om[k]);
                }
            }
        }
        load_unit(cur, next_unit());
    };
    // Finishes `count` <= 64 parked queries, records [first, first + count) of the queue.
    auto drain = [&](uint32_t first, uint32_t count) {
        // The records, and the "nothing feasible" stored for these queries by the main loop, must
        // have left this wavefront before they are read back and overwritten.  Writer and reader are
        // the same wavefront, so workgroup scope is enough (a wider release would write back L2).
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
        const bool have = (uint32_t)lane < count;
        const int32_t *e = (const int32_t *)(wq + first + (have ? lane : 0));
        int32_t qi = __hip_atomic_load(e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        v4i side{-1, 0, 0, 3};   // last pass of the complete Case I: what the first tier suggests, and how far that is
        if (kCase1 && kSecond) {
            const int32_t r = have ? qi : 0;
            qi = open_in[r].x;
            side = ((const v4i *)q.open_side + (int64_t)blockIdx.x * q.open_cap)[r];
        }
        const int32_t slo = __hip_atomic_load(e + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        const int32_t min_acc = __hip_atomic_load(e + 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        const int32_t s_ld = __hip_atomic_load(e + 3, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        const bool final_miss = kSuggest && have && ((uint32_t)s_ld & kParkFinal);
        const uint32_t s = have ? ((uint32_t)s_ld & ~kParkFinal) : (uint32_t)tv.S;   // idle lanes: the empty slice
        const v2u h = lmem.ld64(lds_hdr0 + s * kLdsHdrBytes);
        const bool resident = !(h.y & kHdrPark);
        const uint32_t lbody = h.x & ((1u << kLdsAddrBits) - 1u);
        uint32_t y = h.y, rec = h.y & 0xFFFFu, gbody = 0;
        if (__ballot(!resident)) {   // slices without a body in LDS: header from global memory
            const uint4 g = ix.hdr[resident ? (uint32_t)tv.S : s];
            if (!resident) { y = g.y; rec = g.z; gbody = g.x; }
        }
        const bool indexed = !(y & kHdrPark);
        const uint32_t keys0 = (y >> kHdrK0Shift) & 0x3Fu, keys1 = (y >> kHdrK1Shift) & 0x3Fu;   // Re of the bodies
        const uint32_t size0 = body_bytes(keys0);
        const uint32_t dd[1] = {acc_threshold(min_acc, acc_base_m1)}, lim[1] = {(uint32_t)slo};
        int32_t ans = -1, wk = -1;
        auto take_step = [&](uint32_t at) {   // the answer is step `at` of the index
            ans = ix.step_row[at];
            if (kWorker) wk = ix.step_worker[at];
        };
        bool done = final_miss;
        // bodies in global memory (the first one only if the main loop could not use an LDS copy):
        // both are searched together, level by level, so that one body's trips to memory hide the other's
        const bool need_g0 = have && indexed && !resident && !done;
        const bool need_g1 = have && indexed && keys1 != 0u && !resident && !done;
        if (__ballot(need_g0 | need_g1)) {
            const uint32_t bd[2] = {need_g0 ? gbody : 0u, need_g1 ? gbody + size0 : 0u};
            const uint32_t ks[2] = {need_g0 ? keys0 : 2u, need_g1 ? keys1 : 2u};
            const uint32_t dd2[2] = {dd[0], dd[0]}, lim2[2] = {lim[0], lim[0]};
            uint32_t m[2];
            search_bodies<2>(gmem, nit, bd, ks, dd2, lim2, m);
            const bool hit0 = need_g0 && m[0], hit1 = need_g1 && !hit0 && m[1];
            if (hit0) take_step(rec + __builtin_ctz(m[0]));
            if (hit1) take_step(rec + kBodySteps + __builtin_ctz(m[1]));
            done = done || hit0 || hit1;
            st_global += (uint32_t)__builtin_popcountll(__ballot(hit0));
            st_second += (uint32_t)__builtin_popcountll(__ballot(hit1));
        }
        // second body of a slice whose bodies are in LDS
        const bool need_l1 = have && indexed && keys1 != 0u && resident && !done;
        if (__ballot(need_l1)) {
            const uint32_t bd[1] = {need_l1 ? lbody + size0 : rebase}, ks[1] = {need_l1 ? keys1 : 2u};
            uint32_t m[1];
            search_bodies<1>(lmem, nit, bd, ks, dd, lim, m);
            if (need_l1 && m[0]) { take_step(rec + kBodySteps + __builtin_ctz(m[0])); done = true; }
            st_second += (uint32_t)__builtin_popcountll(__ballot(need_l1 && m[0]));
        }
        // no body, or both bodies missed and more steps exist: scan the slice in rank order
        uint64_t todo = __ballot(have && !done && (!indexed || (y & kHdrTrunc)));
        if (todo) {
            st_scanned += (uint32_t)__builtin_popcountll(todo);
            const int32_t task = (int32_t)(s / (uint32_t)tv.B), bidx = (int32_t)(s - (uint32_t)task * (uint32_t)tv.B);
            while (todo) {
                const int l = __builtin_ctzll(todo);
                todo &= todo - 1;
                const int32_t t = __builtin_amdgcn_readlane(task, l), b = __builtin_amdgcn_readlane(bidx, l);
                const int32_t am = __builtin_amdgcn_readlane(min_acc, l);
                const uint32_t bound = (uint32_t)__builtin_amdgcn_readlane(slo, l);
                const int32_t seg = tv.seg_off[t], L = tv.seg_len[t];
                const int64_t col = (int64_t)b * tv.Vp + seg;
                int32_t found = -1;
                for (int32_t blk = 0; blk < L; blk += 64) {
                    const int32_t pos = blk + lane;
                    const bool ok = pos < L && tv.acc_r[col + pos] >= am && tv.tot_r[col + pos] <= bound;
                    const uint64_t bm = __ballot(ok);
                    if (bm) { found = blk + (int32_t)__builtin_ctzll(bm); break; }
                }
                if (lane == l) {
                    ans = found >= 0 ? tv.orig_r[col + found] : -1;
                    if (kWorker) wk = found >= 0 ? q.row_worker[ans] : -1;
                }
            }
        }
        st_none += (uint32_t)__builtin_popcountll(__ballot(have && !final_miss && ans < 0));
        if (kSecond) {
            if (have && ans >= 0) {
                q.out[qi] = ans; q.tier[qi] = 2;
                if (kCase1) q.closest[qi] = ans;
                if (kWorker) q.worker[qi] = wk;
            }
        } else if (have && !final_miss) {
            q.out[qi] = ans;
        }
        uint32_t open_at = 0;   // first tier: where this lane's query went in the workgroup's list
        if (kFirst) {   // the main loop has stored tier 0 for a parked query
            if (have && ans >= 0) {
                q.tier[qi] = 1;
                if (kWorker) q.worker[qi] = wk;
            }
            const uint64_t om = __ballot(have && ans < 0);
            if (om) {
                open_at = open_room((uint32_t)__builtin_popcountll(om)) + lanes_below(om);
                if (have && ans < 0) open_out[open_at] = v4i{qi, slo, min_acc, (int32_t)s};
            }
        }
        if (kSuggest) {
            // the suggestion for the queries that ended with nothing feasible
            const bool open = have && ans < 0;
            const bool by_index = open && indexed && !(y & kHdrTrunc);
            int32_t sug = ans;
            HowFar mine{3, 0, 0};   // how far the suggestion is from the requirements
            const bool in_lds = by_index && resident, in_mem = by_index && !resident;
            if (__ballot(in_lds)) {
                const ClosestStep c = closest_step(lmem, nit, in_lds ? lbody : rebase, in_lds ? keys0 : 2u,
                                                   in_lds ? keys1 : 0u, dd[0], slo, min_acc, acc_base_m1);
                if (in_lds && c.step >= 0) { sug = ix.step_row[rec + (uint32_t)c.step]; mine = c.how; }
            }
            if (__ballot(in_mem)) {
                const ClosestStep c = closest_step(gmem, nit, in_mem ? gbody : 0u, in_mem ? keys0 : 2u,
                                                   in_mem ? keys1 : 0u, dd[0], slo, min_acc, acc_base_m1);
                if (in_mem && c.step >= 0) { sug = ix.step_row[rec + (uint32_t)c.step]; mine = c.how; }
            }
            // slices without a complete index: the whole slice, in rank order, by the wavefront
            uint64_t rest = __ballot(open && !by_index);
            if (rest) {
                const int32_t task = (int32_t)(s / (uint32_t)tv.B), bidx = (int32_t)(s - (uint32_t)task * (uint32_t)tv.B);
                while (rest) {
                    const int l = __builtin_ctzll(rest);
                    rest &= rest - 1;
                    const int32_t t = __builtin_amdgcn_readlane(task, l), b = __builtin_amdgcn_readlane(bidx, l);
                    const int64_t am = __builtin_amdgcn_readlane(min_acc, l), bound = __builtin_amdgcn_readlane(slo, l);
                    HowFar how;
                    const int32_t found = closest_by_scan(tv, t, b, am, bound, lane, &how);
                    if (lane == l) { sug = found; mine = how; }
                }
            }
            if (kCase1 && kFirst && open)   // for the second tier: this tier's suggestion and how far it is
                ((v4i *)q.open_side + (int64_t)blockIdx.x * q.open_cap)[open_at] = pack_side(sug, mine);
            if (kCase1 && kSecond) {
                // the closer of the two tiers' suggestions, by (requirements missed, latency beyond the
                // bound, accuracy below the bound), the first tier's at a tie; q.closest holds the first tier's
                if (open && sug >= 0) {
                    const bool keep_first = side.x >= 0 && closer_or_equal(unpack_side(side), mine);
                    if (!keep_first) q.closest[qi] = sug;
                }
            } else if (have) {
                q.closest[qi] = sug;
            }
        }
    };

    {
        // The rotation is interrupted only when 64 parked queries have collected (one full pass of
        // the wavefront) and resumed where it stopped.
        int phase = 0;
        bool more = true;
        while (more) {
            for (;;) {
                if (phase == 0) {
                    if (fa.unit < 0) { more = false; break; }
                    stage(fa);
                    phase = 1;
                    if (cnt >= 64u) break;
                }
                if (fb.unit < 0) { more = false; break; }
                stage(fb);
                phase = 0;
                if (cnt >= 64u) break;
            }
            store_unit();   // a parked query gets -1 here and its real answer in drain()
            p_i0 = -1;
            while (cnt >= 64u || (!more && cnt > 0u)) {
                const uint32_t c = cnt < 64u ? cnt : 64u;
                drain(cnt - c, c);
                cnt -= c;
            }
        }
    }
    // statistics of this launch, per workgroup (plain stores: nothing waits for them)
    if (lane == 0) {
        const uint32_t st[kLookupStats] = {st_parked, st_second, st_global, st_scanned, st_none};
#pragma unroll
        for (int i = 0; i < kLookupStats; ++i)
            if (st[i]) atomicAdd(&lds_w[4 + i], st[i]);
    }
    __syncthreads();
    if (tid < kLookupStats) ix.stats[blockIdx.x * kLookupStats + tid] = lds_w[4 + tid];
    if (blockIdx.x == 0 && tid == 0) ix.stats[-1] = gridDim.x;
    if (kFirst && tid == 0) q.open_count[blockIdx.x] = (int32_t)s_open;
}

}  // namespace

// ---------------------------------------------------------------- launchers

namespace {

template <bool kTwo>
hipError_t launch_build(const TableView &ta, const IndexView &ia, const TableView &tb, const IndexView &ib, hipStream_t st,
                        const LaunchEvents *ev)
{
    constexpr unsigned tables = kTwo ? 2 : 1;
    if (ta.S <= 0) return hipSuccess;
    const dim3 block(64 * kBuildWaves);
    // One slice per workgroup as long as all of them are on the device at once (four workgroups of these registers
    // to each of 256 compute units; the sums over the slices before are short, too).  us for one slice per workgroup / per
    // wavefront: 160 slices of 45 entries 7.3 / 9.9, 400 of 2000 15.9 / 21, 600 of 60 on average 15.9 / 24.4; two tables
    // of 800 slices of 200 20.3 / 12.7; 1600 of 60 16.0 / 13.5.  Without groups only up to 512: an index of more
    // slices mostly outgrows the lookup's LDS mirror, and in the order of the slices' numbers, not of their arrival (short
    // staircases first), more slices stay outside (1M queries on 800 slices 13.5 us against 12.7, which the
    // build's 11.5 against 15.1 does not make up for: there are more batches than reports).
    if ((int64_t)ta.S * tables <= 1024 && (ta.S <= 512 || ia.num_groups > 1)) {
        const dim3 each((unsigned)ta.S, tables);
        if (ta.max_len <= 256) return launch_kernel(ev, k_index_build_shared<1, kTwo>, each, block, 0, st, ta, ia, tb, ib);
        if (ta.max_len <= 512) return launch_kernel(ev, k_index_build_shared<2, kTwo>, each, block, 0, st, ta, ia, tb, ib);
        if (ta.max_len <= 1024) return launch_kernel(ev, k_index_build_shared<4, kTwo>, each, block, 0, st, ta, ia, tb, ib);
        return launch_kernel(ev, k_index_build_shared<8, kTwo>, each, block, 0, st, ta, ia, tb, ib);
    }
    const dim3 grid((unsigned)((ta.S + kBuildWaves - 1) / kBuildWaves), tables);
    // no slice longer than one chunk: a chunk of that size, whose loops have no idle rounds (us, two tables of 100
    // tasks of 200 variants x 8: 13.5 with chunks of 4 x 64 entries, 13.7 with 8, 14.7 with 16)
    if (ta.max_len <= 256) return launch_kernel(ev, k_index_build<4, kTwo>, grid, block, 0, st, ta, ia, tb, ib);
    if (ta.max_len <= 512) return launch_kernel(ev, k_index_build<8, kTwo>, grid, block, 0, st, ta, ia, tb, ib);
    // up to 1024 slices, of which some are longer than that: chunks of twice the size, one round of the filter instead of
    // two for 2048 entries (us, load report and build: 800 slices of 1100 / 1500 entries 29.5 / 32.7 -> 26.1 / 28.2, 1000 slices
    // of up to 13,396 entries 102 -> 72).  With more slices, or two tables (of more than 512 slices, or they would not be
    // here), fewer workgroups at a time cost more than that (two tables of 800 slices of 1500: 30.3 -> 34.2).
    if constexpr (!kTwo)
        if (ta.S <= 1024 && ta.max_len > 1024) return launch_kernel(ev, k_index_build<32, kTwo>, grid, block, 0, st, ta, ia, tb, ib);
    return launch_kernel(ev, k_index_build<16, kTwo>, grid, block, 0, st, ta, ia, tb, ib);
}

}  // namespace

hipError_t launch_index_build(const TableView &tv, const IndexView &ix, hipStream_t st, const LaunchEvents *ev)
{
    return launch_build<false>(tv, ix, tv, ix, st, ev);
}

hipError_t launch_index_build(const TableView &ta, const IndexView &ia, const TableView &tb, const IndexView &ib, hipStream_t st,
                              const LaunchEvents *ev)
{
    return launch_build<true>(ta, ia, tb, ib, st, ev);
}

int index_select_blocks(int num_cus) { return num_cus; }
int index_stat_blocks(int num_cus) { return kStatShare * num_cus; }

// Records per workgroup of the lists a first-tier pass over n queries may write: every query of
// the workgroup's share of the units.
int32_t index_open_cap(int32_t n, int num_cus)
{
    const int64_t unit = 64 * kPerThread, blocks = index_select_blocks(num_cus);
    const int64_t nunits = (n + unit - 1) / unit;
    return (int32_t)(((nunits + blocks - 1) / blocks) * unit);
}

size_t index_park_bytes(int num_cus)
{
    return (size_t)index_select_blocks(num_cus) * (kSelThreads / 64) * kWaveQueue * sizeof(v4i);
}

hipError_t launch_index_select(const TableView &tv, const IndexView &ix, const QueryView &q,
                               int32_t *park_mem, uint32_t lds_bytes, int num_cus, hipStream_t st, const LaunchEvents *ev)
{
    const int blocks = index_select_blocks(num_cus);
    const uint32_t fixed = kLdsCtrlBytes + lds_header_bytes(tv.S);
    if (lds_bytes <= fixed) return hipErrorInvalidValue;   // (no mirror: nothing sends a call here)
    lds_bytes = fixed + ((lds_bytes - fixed) & ~15u);
    auto kernel = q.pass == 1 ? k_index_select<1> : q.pass == 2 ? k_index_select<2> : q.pass == 3 ? k_index_select<3> :
                  q.pass == 4 ? k_index_select<4> : q.pass == 5 ? k_index_select<5> : q.pass == 6 ? k_index_select<6> :
                  q.pass == 7 ? k_index_select<7> : q.pass == 8 ? k_index_select<8> : q.pass == 9 ? k_index_select<9> : k_index_select<0>;
    hipError_t e = hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)lds_bytes);
    if (e != hipSuccess) return e;
    // the worker modes keep the 16-bit workers of the hot steps behind the bodies
    uint32_t hot = 0;
    const bool worker_pass = q.pass == 4 || q.pass == 5 || q.pass == 8 || q.pass == 9;
    if (worker_pass && ix.hot_worker) hot = ((uint32_t)tv.S * ix.hot_rows * 2u + 15u) & ~15u;
    if (hot + 1024u > lds_bytes - fixed) hot = 0;   // (never with a sensible table; the kernel then must not look for them)
    IndexView ixk = ix;
    if (!hot) ixk.hot_worker = nullptr;
    return launch_kernel(ev, kernel, dim3((unsigned)blocks), dim3((unsigned)kSelThreads), lds_bytes, st, tv, ixk, q,
                         park_mem, lds_bytes - fixed - hot);
}

}  // namespace infaas
