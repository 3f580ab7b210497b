// Device helpers shared by the lookup kernels: readers of index memory and the search of a body.
#pragma once

#include "internal.h"

namespace infaas {
namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef uint32_t v2u __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t lanes_below(uint64_t mask)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                     __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

#define INFAAS_LDS __attribute__((address_space(3)))

// Workgroup barrier that orders LDS traffic only: what the wavefronts have written to LDS is visible
// to each other behind it, while their requests to global memory stay in flight (__syncthreads also
// waits for those -- for an atomic on a contended word, microseconds).
__device__ __forceinline__ void lds_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}


// Readers of index memory by 32-bit byte address: an LDS address, or an offset from a global base.
struct LdsMem {
    __device__ __forceinline__ uint32_t ld32(uint32_t a, uint32_t imm) const { return *(const INFAAS_LDS uint32_t *)(a + imm); }
    __device__ __forceinline__ uint32_t ld16(uint32_t a, uint32_t imm) const { return *(const INFAAS_LDS uint16_t *)(a + imm); }
    __device__ __forceinline__ v2u ld64(uint32_t a) const { return *(const INFAAS_LDS v2u *)a; }
};
struct GlobalMem {
    const uint8_t *p;
    __device__ __forceinline__ uint32_t ld32(uint32_t a, uint32_t imm) const { return *(const uint32_t *)(p + a + imm); }
    __device__ __forceinline__ uint32_t ld16(uint32_t a, uint32_t imm) const { return *(const uint16_t *)(p + a + imm); }
};

// First fitting step of kN bodies (one per query of this lane), as bit sets; the kN searches are
// interleaved so that their dependent reads overlap.  Branch-free apart from the wave-uniform
// probe count.  body[k] / re[k]: address and keys per array (Re) of the body; dd[k]: accuracy
// threshold in key space; lim[k]: latency bound.
template <int kN, class Mem>
__device__ __forceinline__ void search_bodies(const Mem &mem, int nit, const uint32_t (&body)[kN],
                                              const uint32_t (&re)[kN], const uint32_t (&dd)[kN],
                                              const uint32_t (&lim)[kN], uint32_t (&m)[kN])
{
    uint32_t pa[kN], la[kN], pt[kN], lt[kN];
#pragma unroll
    for (int k = 0; k < kN; ++k) {
        pa[k] = body[k];                       // accuracy key j (1-based) at body + 2 + 2j
        la[k] = body[k] + 2u * re[k];          // probes beyond the keys land on the last sentinel
        pt[k] = la[k];                         // latency key j at body + 2 Re + 4j
        lt[k] = pt[k] + 4u * re[k];
    }
#pragma unroll
    for (int it = 4; it >= 0; --it) {
        if (it < nit) {
            uint32_t ca[kN], ct[kN], ka[kN], kt[kN];
#pragma unroll
            for (int k = 0; k < kN; ++k) {   // all reads of a level first, so that they overlap
                ca[k] = pa[k] + (2u << it);
                ct[k] = pt[k] + (4u << it);
                ka[k] = mem.ld16(ca[k] < la[k] ? ca[k] : la[k], 2u);
                kt[k] = mem.ld32(ct[k] < lt[k] ? ct[k] : lt[k], 0u);
            }
#pragma unroll
            for (int k = 0; k < kN; ++k) {
                pa[k] = ka[k] >= dd[k] ? ca[k] : pa[k];
                pt[k] = kt[k] <= lim[k] ? ct[k] : pt[k];
            }
        }
    }
#pragma unroll
    for (int k = 0; k < kN; ++k) {
        // A[p] at body + 4 + 6 Re + 4p with pa = body + 2p;  S[ps] at body + 4 + 10 Re + 4 ps with
        // pt = body + 2 Re + 4 ps
        const uint32_t a_at = 2u * pa[k] + (6u * re[k] - body[k]);
        const uint32_t s_at = pt[k] + 8u * re[k];
        m[k] = mem.ld32(a_at, 4u) & mem.ld32(s_at, 4u);
    }
}

// The closest variant of slice (t, b) for a query that nothing satisfies, by the whole wavefront over
// the whole slice in rank order: first by (requirements missed, latency beyond `bound`, accuracy
// below `am`), the earlier rank at a tie.  Entries of a table that serves one state which belong to
// variants of other states (latency key all ones) are passed over.  Returns the caller's row, the
// same in every lane, or -1 when the slice has no entry to offer; *how gets its distance.
struct HowFar {
    int32_t missed;          // of the two requirements
    int64_t over, shortf;    // latency beyond the bound, accuracy below the bound (0 when met)
};
// (requirements missed, latency beyond the bound, accuracy below the bound): the smaller, the closer
__device__ __forceinline__ bool closer_or_equal(const HowFar &a, const HowFar &b)
{
    return a.missed < b.missed || (a.missed == b.missed && (a.over < b.over || (a.over == b.over && a.shortf <= b.shortf)));
}
__device__ __forceinline__ int32_t closest_by_scan(const TableView &tv, int32_t t, int32_t b, int64_t am, int64_t bound, int lane,
                                                   HowFar *how = nullptr)
{
    const int32_t seg = tv.seg_off[t], L = tv.seg_len[t];
    const int64_t col = (int64_t)b * tv.Vp + seg;
    // per lane the best of its entries, earlier rank first
    int32_t b_missed = 3, b_pos = 0x7FFFFFFF;
    int64_t b_over = 0, b_short = 0;
    for (int32_t pos = lane; pos < L; pos += 64) {
        const int64_t tt = (int64_t)tv.tot_r[col + pos], a = (int64_t)tv.acc_r[col + pos];
        const int64_t over = tt > bound ? tt - bound : 0, shortf = a < am ? am - a : 0;
        const int32_t missed = (over > 0) + (shortf > 0);
        const bool masked = tv.state != nullptr && tt == 0xFFFFFFFFll;   // a variant of another state
        const bool better = !masked && (missed < b_missed || (missed == b_missed && (over < b_over ||
                            (over == b_over && shortf < b_short))));
        if (better) { b_missed = missed; b_over = over; b_short = shortf; b_pos = pos; }
    }
    for (int off = 32; off; off >>= 1) {   // then the best of the wavefront
        const int32_t o_missed = __shfl_xor(b_missed, off), o_pos = __shfl_xor(b_pos, off);
        const int64_t o_over = __shfl_xor(b_over, off), o_short = __shfl_xor(b_short, off);
        const bool better = o_missed < b_missed || (o_missed == b_missed && (o_over < b_over ||
                            (o_over == b_over && (o_short < b_short || (o_short == b_short && o_pos < b_pos)))));
        if (better) { b_missed = o_missed; b_over = o_over; b_short = o_short; b_pos = o_pos; }
    }
    if (how) { how->missed = b_missed; how->over = b_over; how->shortf = b_short; }
    return b_missed < 3 ? tv.orig_r[col + b_pos] : -1;
}

// The first entry, in rank order, of the slice with rank_hdr entry `rh` that fits (min_acc, bound), as the
// caller's row or -1; one query per lane (entry S: no query), for slices whose TableView::rank_nodes the index build has written.
// "The accuracy has come up to min_acc and the latency down to bound" turns true once along a slice and
// stays true, so the first 16 entries that can hold the answer are found by descending the levels, one
// node each.  Four lanes read a query's node together (64 bytes at a time, which is what the L1 delivers in
// a cycle), so that a level costs one line of memory where a bisection by the lane itself would cost up to
// four.  Those 16 entries are tried in the same manner.  Where accuracy rises and latency falls with the
// rank the answer is among them.  What is still open goes on from there, the whole wavefront on one query
// after the other: all of it where that is 512 entries or fewer, else the rest of the block of 256, then the sorted
// blocks, eight at a time, which tell exactly whether they hold an entry that fits, then the first one that does.
// 16M queries on 50 tasks of 2000 variants none of which dominates another: 0.55 ms; the same with the lane's own
// bisection over a running extreme per entry 1.32 ms, with eight lanes to a node instead of four as fast (and 41 us
// instead of 25 for 1.4M queries on tasks of 81 variants).  Without the sorted blocks the two families of
// use_ranked() (api.hip) took 3.1 ms per 4M queries instead of 1.2.  What bounds it is scattered reads of L2 lines,
// two levels, two columns, a row and two headers per query.  (Comparisons are combined with & and |: with && the
// 16-byte reads are split into dwords behind branches, 0.62 ms instead of 0.55.)
// kAhead false: with fewer registers, for kernels that have the search beside much else.
template <bool kAhead>
__device__ __forceinline__ int32_t ranked_first_fit(const TableView &tv, const uint4 &rh, int32_t min_acc, uint32_t bound)
{
    const int lane = threadIdx.x & 63, sub = lane & 3, round = lane >> 4;
    const int back = 4 * (lane & 15);            // where this lane's query is answered in its round
    const int32_t L = (int32_t)rh.y;
    int32_t am[4];       // of the query this lane works for in round r
    uint32_t bd[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        am[r] = __shfl(min_acc, 16 * r + (lane >> 2));
        bd[r] = (uint32_t)__shfl((int)bound, 16 * r + (lane >> 2));
    }
    auto quad = [](int v, int o) {   // the value of the lane 1 or 2 away inside the four
        return o == 1 ? __builtin_amdgcn_mov_dpp(v, 0xB1, 0xF, 0xF, true) : __builtin_amdgcn_mov_dpp(v, 0x4E, 0xF, 0xF, true);
    };
    int top = 1;   // this lane's highest level
    while (level_nodes(L, top) > 1) ++top;
    bool open = L > 0;
    int32_t node = 0;
    int level = 1;
    while (__ballot(open && top > level)) ++level;   // the highest of all lanes
    for (; level >= 1; --level) {
        const bool here = open && level <= top;
        uint32_t at = rh.z;
        for (int i = 1; i < level; ++i) at += (uint32_t)level_nodes(L, i);
        at = here ? at + (uint32_t)node : 0u;
        int cnt = 0;   // pairs of the node that do not meet the requirements yet: they come first
        uint4 v[4][2];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const uint4 *p = tv.rank_nodes() + (uint64_t)(uint32_t)__shfl((int)at, 16 * r + (lane >> 2)) * 8u + (uint32_t)sub;
            v[r][0] = p[0];
            v[r][1] = p[4];
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            int c = 0;
#pragma unroll
            for (int k = 0; k < 2; ++k)
                c += (int)(((int32_t)v[r][k].x < am[r]) | (v[r][k].y > bd[r])) + (int)(((int32_t)v[r][k].z < am[r]) | (v[r][k].w > bd[r]));
            c += quad(c, 1);
            c += quad(c, 2);
            c = __shfl(c, back);
            cnt = round == r ? c : cnt;
        }
        if (here) {
            node = node * 16 + cnt;
            open = level == 1 ? (int64_t)node * 16 < L : (cnt < 16 && node < level_nodes(L, level - 1));
        }
    }
    int32_t found = -1, from = node * 16;
    {   // the 16 entries
        const uint32_t at = open ? rh.x + ((uint32_t)from >> 2) : 0u;
        const int32_t left = open ? L - from : 0;
        uint4 a[4], w[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const uint64_t p = (uint64_t)(uint32_t)__shfl((int)at, 16 * r + (lane >> 2)) + (uint32_t)sub;
            a[r] = ((const uint4 *)tv.acc_r)[p];
            w[r] = ((const uint4 *)tv.tot_r)[p];
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            uint32_t m = 0x10000u;
            m |= (((int32_t)a[r].x >= am[r]) & (w[r].x <= bd[r])) ? 1u : 0u;
            m |= (((int32_t)a[r].y >= am[r]) & (w[r].y <= bd[r])) ? 2u : 0u;
            m |= (((int32_t)a[r].z >= am[r]) & (w[r].z <= bd[r])) ? 4u : 0u;
            m |= (((int32_t)a[r].w >= am[r]) & (w[r].w <= bd[r])) ? 8u : 0u;
            int f = 4 * sub + __builtin_ctz(m), o = quad(f, 1);   // 16 or more: none of this lane's four
            f = o < f ? o : f;
            o = quad(f, 2);
            f = o < f ? o : f;
            f = __shfl(f, back);
            if (round == r && f < 16 && f < left) found = from + f;
        }
        open = open && found < 0 && left > 16;
        from += 16;
    }
    uint64_t todo = __ballot(open);
    while (todo) {
        const int l = __builtin_ctzll(todo);
        todo &= todo - 1;
        const int32_t lo = __builtin_amdgcn_readlane(from, l), len = __builtin_amdgcn_readlane(L, l);
        const int32_t qa = __builtin_amdgcn_readlane(min_acc, l);
        const uint32_t qb = (uint32_t)__builtin_amdgcn_readlane((int)bound, l);
        const int64_t c = (int64_t)(uint32_t)__builtin_amdgcn_readlane((int)rh.x, l) * 4;
        // the first of the entries first + 4 * lane + {0, 1, 2, 3} below hi that fits, or -1 (first: a multiple of 4).
        // (Slices start at multiples of 4 and are padded to multiples of 4 with entries that never fit.)
        auto first_fit = [&](const uint4 &a, const uint4 &w, int32_t first, int32_t hi) -> int32_t {
            uint32_t m = 0;
            m |= (((int32_t)a.x >= qa) & (w.x <= qb)) ? 1u : 0u;
            m |= (((int32_t)a.y >= qa) & (w.y <= qb)) ? 2u : 0u;
            m |= (((int32_t)a.z >= qa) & (w.z <= qb)) ? 4u : 0u;
            m |= (((int32_t)a.w >= qa) & (w.w <= qb)) ? 8u : 0u;
            m = first + 4 * lane < hi ? m : 0u;
            const uint64_t any = __ballot(m != 0u);
            if (!any) return -1;
            const int f = __builtin_ctzll(any);
            return first + 4 * f + __builtin_ctz((uint32_t)__builtin_amdgcn_readlane((int)m, f));
        };
        auto try_block = [&](int32_t first, int32_t hi) -> int32_t {   // at most 256 entries
            const int64_t at = c + (first + 4 * lane < hi ? first + 4 * lane : 0);
            return first_fit(*(const uint4 *)(tv.acc_r + at), *(const uint4 *)(tv.tot_r + at), first, hi);
        };
        // All that is left at once: two rounds of reads instead of up to four.  (1M queries most of which have no answer,
        // 300 entries of random accuracy and latency to a slice: 337 us block by block, 111 so, 297 with the scan engine.)
        if (kAhead && len - lo > 256 && len - lo <= kRankAtOnce) {
            const int64_t at0 = c + (lo + 4 * lane < len ? lo + 4 * lane : 0), at1 = c + (lo + 256 + 4 * lane < len ? lo + 256 + 4 * lane : 0);
            const uint4 a0 = *(const uint4 *)(tv.acc_r + at0), w0 = *(const uint4 *)(tv.tot_r + at0);
            const uint4 a1 = *(const uint4 *)(tv.acc_r + at1), w1 = *(const uint4 *)(tv.tot_r + at1);
            int32_t hit = first_fit(a0, w0, lo, len);
            hit = hit < 0 ? first_fit(a1, w1, lo + 256, len) : hit;
            if (lane == l) found = hit;
            continue;
        }
        if (len - lo <= kRankAtOnce) {
            int32_t hit = -1;
            for (int32_t first = lo; hit < 0 && first < len; first += 256) hit = try_block(first, first + 256 < len ? first + 256 : len);
            if (lane == l) found = hit;
            continue;
        }
        int32_t end = (lo + kRankBlock - 1) & ~(kRankBlock - 1);
        int32_t hit = lo < end ? try_block(lo, end < len ? end : len) : -1;
        const int32_t nblk = rank_blocks(len);
        const uint32_t sorted = (uint32_t)__builtin_amdgcn_readlane((int)rh.z, l) + (uint32_t)all_level_nodes(len);
        for (int32_t b0 = end / kRankBlock; hit < 0 && b0 < nblk; b0 += 8) {
            const int32_t blk = b0 + (lane >> 3);
            const bool in = blk < nblk;
            const uint4 *p = tv.rank_nodes() + ((uint64_t)sorted + (uint64_t)(in ? blk : b0) * kRankBlockNodes) * 8u + (uint32_t)(lane & 7);
            const uint4 v = *p;   // of the last pair of each node: is the node altogether accurate enough?
            const bool k0 = (int32_t)v.x >= qa, k1 = (int32_t)v.z >= qa;
            const uint64_t n0 = __ballot(k0), n1 = __ballot(k1);
            const int whole = __builtin_popcount((uint32_t)(n0 >> (lane & 56)) & 0xFFu) + __builtin_popcount((uint32_t)(n1 >> (lane & 56)) & 0xFFu);
            const uint4 u = p[8 * (whole < 16 ? 1 + whole : 16)];
            bool fits = (k0 & (v.y <= qb)) | (k1 & (v.w <= qb));
            fits = fits | (((int32_t)u.x >= qa) & (u.y <= qb)) | (((int32_t)u.z >= qa) & (u.w <= qb));
            const uint64_t any = __ballot(fits && in);
            if (any) {
                const int32_t first = (b0 + (__builtin_ctzll(any) >> 3)) * kRankBlock;
                hit = try_block(first, first + kRankBlock < len ? first + kRankBlock : len);
                break;
            }
        }
        if (lane == l) found = hit;
    }
    return found >= 0 ? tv.orig_r[(int64_t)rh.x * 4 + found] : -1;
}

// ---- lines (internal.h)

// What a query is compared with in a line: {accuracy threshold, shifted like the keys; latency bound}.
__device__ __forceinline__ uint32_t line_threshold(const IndexView &ix, int32_t min_acc, int32_t acc_base_m1)
{
    const int32_t d = __builtin_elementwise_sub_sat(min_acc, acc_base_m1);   // keys are accuracy - acc_base_m1 >= 1
    const int32_t top = (int32_t)ix.line_top;
    return (uint32_t)(d < 1 ? 1 : d > top ? top : d) << ix.line_shift();
}
// What a line says to a query (lookup_lines): the entry that answers it, {number of the lane that had it << 30 | row}, or one of the
// codes from kCodeOpen on, in this order: the next line may, kCodeRank, nothing does.
constexpr uint32_t kCodeOpen = 0xE0000000u, kCodeRank = 0xFFFFFFFDu, kCodeNone = 0xFFFFFFFEu;
__device__ __forceinline__ bool line_open(uint32_t code) { return code >= kCodeOpen && code < kCodeRank; }
template <int kLane>
__device__ __forceinline__ uint32_t of_quad(uint32_t v)   // the value of one of the four lanes of a quad
{
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, kLane * 0x55, 0xF, 0xF, true);
}
// What a line says, of which this lane has four entries, for the four lanes of its quad.  tag: the lane's number in the quad << 30;
// shift: 3 in the last of the four, else 31.
__device__ __forceinline__ uint32_t line_says(const uint4 &w0, const uint4 &w1, uint32_t d, uint32_t l, uint32_t row_mask, uint32_t tag, uint32_t shift)
{
    const bool f0 = (w0.x >= d) & (w0.y <= l), f1 = (w0.z >= d) & (w0.w <= l);
    const bool f2 = (w1.x >= d) & (w1.y <= l), f3 = (w1.z >= d) & (w1.w <= l);
    uint32_t word = f2 ? w1.x : w1.z;   // the first of the lane's four that fits
    word = f1 ? w0.z : word;
    word = f0 ? w0.x : word;
    uint32_t mine = (word & row_mask) | tag;
    // nothing fits: the last lane's last entry tells what follows (a step: a code between kCodeOpen and kCodeRank, kLineEnd: all
    // ones); the other lanes say nothing (all ones, or one less)
    mine = (f0 | f1 | f2 | f3) ? mine : __builtin_amdgcn_alignbit(~0u, w1.w, shift);
    uint32_t o = (uint32_t)__builtin_amdgcn_mov_dpp((int)mine, 0xB1, 0xF, 0xF, true);
    mine = o < mine ? o : mine;
    o = (uint32_t)__builtin_amdgcn_mov_dpp((int)mine, 0x4E, 0xF, 0xF, true);
    return o < mine ? o : mine;
}
// One query per lane: the line at byte `at` of `lines`, threshold d, latency bound l.  In round r the four lanes of every quad read the
// line of the query of the r-th of them and compare it with all 16 entries, four to a lane.  `rounds`, where kSome is set: bit r
// clear: none of the queries of round r is looked at (their code is 0).
// Bound by the lines: a random one from L2 costs 4.5 ps on the whole card, 3.6 from L1 (quads that read two times 64 bytes and do nothing else);
// 24 vector instructions to a round, 95 per 64 queries with what precedes and follows, are 2.4.
template <bool kSome>
__device__ __forceinline__ uint32_t lookup_lines(const uint8_t *lines, uint32_t at, uint32_t d, uint32_t l, uint32_t row_mask, uint32_t rounds = 15u)
{
    const uint32_t sub = threadIdx.x & 3u, tag = sub << 30, shift = sub == 3u ? 3u : 31u;
    uint4 v[4][2];
    uint32_t code = 0u;
    auto request = [&](uint4 (&w)[2], uint32_t from) __attribute__((always_inline)) {
        const uint32_t at32 = from + 16u * sub;   // (one 32-bit offset from a uniform base)
        w[0] = *(const uint4 *)(lines + at32);
        w[1] = *(const uint4 *)(lines + at32 + 64);
    };
    auto look = [&](const uint4 (&w)[2], uint32_t dr, uint32_t lr, uint32_t r) __attribute__((always_inline)) {
        const uint32_t mine = line_says(w[0], w[1], dr, lr, row_mask, tag, shift);
        code = sub == r ? mine : code;
    };
    if (!kSome || (rounds & 1u)) request(v[0], of_quad<0>(at));
    if (!kSome || (rounds & 2u)) request(v[1], of_quad<1>(at));
    if (!kSome || (rounds & 4u)) request(v[2], of_quad<2>(at));
    if (!kSome || (rounds & 8u)) request(v[3], of_quad<3>(at));
    if (!kSome || (rounds & 1u)) look(v[0], of_quad<0>(d), of_quad<0>(l), 0u);
    if (!kSome || (rounds & 2u)) look(v[1], of_quad<1>(d), of_quad<1>(l), 1u);
    if (!kSome || (rounds & 4u)) look(v[2], of_quad<2>(d), of_quad<2>(l), 2u);
    if (!kSome || (rounds & 8u)) look(v[3], of_quad<3>(d), of_quad<3>(l), 3u);
    return code;
}
// The lanes of a set, 16 to a round and each of them to a quad, so that a few queries of a wavefront take one round instead of the four
// that they are spread over.  Every lane of the wavefront has to be there.  (us, with the rounds of the lanes and so: complete Case I, 250,001 queries on 50
// tasks of 2000 variants 17.3 / 13.4, 1M on 200 of 60 48.4 / 36.1; suggestions, 300,000 on 100 of 200 14.8 / 11.5.)
struct Packed {
    uint32_t count;   // lanes in the set
    uint32_t place;   // of this lane: among them, or behind them
    uint32_t lane;    // of the one whose place this lane's number is
    __device__ __forceinline__ explicit Packed(uint64_t set)
    {
        const uint32_t me = threadIdx.x & 63u;
        count = (uint32_t)__builtin_popcountll(set);
        place = ((set >> me) & 1u) ? lanes_below(set) : count + lanes_below(~set);
        lane = (uint32_t)__builtin_amdgcn_ds_permute((int)(place * 4u), (int)me);
    }
    // The lane this lane's quad works for in the round that begins with place r0, and of what that quad has found what is this lane's.
    __device__ __forceinline__ int source(uint32_t r0) const { return __shfl((int)lane, (int)(r0 + ((threadIdx.x & 63u) >> 2))); }
    __device__ __forceinline__ uint32_t back(uint32_t v) const { return (uint32_t)__shfl((int)v, (int)(4u * (place & 15u))); }
    __device__ __forceinline__ bool mine(uint32_t r0) const { return place < count && (place >> 4) == (r0 >> 4); }
};
// lookup_lines for the lanes in `set` (the others get kCodeNone, and name the empty line).
__device__ __forceinline__ uint32_t lookup_lines_packed(const uint8_t *lines, uint64_t set, uint32_t at, uint32_t d, uint32_t l, uint32_t row_mask)
{
    const uint32_t sub = threadIdx.x & 3u, tag = sub << 30, shift = sub == 3u ? 3u : 31u;
    const Packed p(set);
    uint32_t code = kCodeNone;
    for (uint32_t r0 = 0; r0 < p.count; r0 += 16u) {
        const int from = p.source(r0);
        const uint32_t at32 = (uint32_t)__shfl((int)at, from) + 16u * sub, dr = (uint32_t)__shfl((int)d, from), lr = (uint32_t)__shfl((int)l, from);
        const uint4 w0 = *(const uint4 *)(lines + at32), w1 = *(const uint4 *)(lines + at32 + 64);
        const uint32_t says = p.back(line_says(w0, w1, dr, lr, row_mask, tag, shift));
        code = p.mine(r0) ? says : code;
    }
    return code;
}
// From the first line's code on: the lines that follow, for the lanes that need them; `plane` gets the plane of the last one looked at.
__device__ __forceinline__ uint32_t follow_lines(const IndexView &ix, uint32_t code, uint32_t s, uint32_t d, uint32_t l, int32_t S, uint32_t &plane)
{
    plane = 0u;
    const uint32_t row_mask = (1u << ix.line_shift()) - 1u;
    for (uint32_t p = 1; p < (uint32_t)kLinePlanes; ++p) {
        const bool more = line_open(code);
        const uint64_t some = __ballot(more);
        if (some == 0ull) break;
        const uint32_t next = lookup_lines_packed(ix.lines, some, (more ? p * ((uint32_t)S + 1u) + s : (uint32_t)S) * kLineBytes, d, l, row_mask);
        code = more ? next : code;
        plane = more ? p : plane;
    }
    return code;
}
// The closest variant of slice s for a query that nothing satisfies (closest_by_scan's order), from the slice's lines, one query per
// lane of those in `want`: its code as lookup_lines gives it, kCodeNone where the slice has nothing to offer, kCodeRank where
// the lines do not hold all of its steps (the closest variant is always a step); how far it is goes to *how.  Where some step is
// within the latency bound it is the most accurate of those; else where some step is accurate enough the fastest of those; else the
// fastest of all, the most accurate among equally fast ones; the earliest at a tie: the smallest of {which of the three, 2 bits; latency, none
// for the first | accuracy from above, 16 bits; place}, by the four lanes of a quad over their entries, then over the lines.
// The first line is in L1 from the selection; bound by the instructions, 100 to a round.
__device__ __forceinline__ uint32_t closest_in_lines(const IndexView &ix, bool want, uint32_t s, int32_t S, uint32_t d, int32_t slo, int32_t min_acc, int32_t acc_base_m1,
                                                     HowFar &how)
{
    const uint32_t sub = threadIdx.x & 3u, shift = sub == 3u ? 3u : 31u, keys = ix.line_shift(), row_mask = (1u << keys) - 1u;
    const uint32_t under = slo < 0 ? 0u : (uint32_t)slo + 1u;   // latencies below this are within the bound
    uint32_t b_hi = ~0u, b_lo = ~0u, b_word = 0u, next = want ? kCodeOpen : kCodeNone;   // the best so far: {order, first word}; what follows
    for (uint32_t p = 0; p < (uint32_t)kLinePlanes; ++p) {
        const uint64_t some = __ballot(line_open(next));
        if (some == 0ull) break;
        const uint32_t at = (line_open(next) ? p * ((uint32_t)S + 1u) + s : (uint32_t)S) * kLineBytes;
        const Packed packed(some);
        uint32_t r_hi = ~0u, r_lo = ~0u, r_word = 0u, r_next = kCodeNone;
        for (uint32_t r0 = 0; r0 < packed.count; r0 += 16u) {
            const int from = packed.source(r0);
            const uint32_t at32 = (uint32_t)__shfl((int)at, from) + 16u * sub, dr = (uint32_t)__shfl((int)d, from), ur = (uint32_t)__shfl((int)under, from);
            const uint4 w0 = *(const uint4 *)(ix.lines + at32), w1 = *(const uint4 *)(ix.lines + at32 + 64);
            const uint32_t first[4] = {w0.x, w0.z, w1.x, w1.z}, tot[4] = {w0.y, w0.w, w1.y, w1.w};
            uint32_t m_hi = ~0u, m_lo = ~0u, m_word = 0u;
            auto take = [&](uint32_t hi, uint32_t lo, uint32_t word) __attribute__((always_inline)) {
                const bool lower = (hi < m_hi) | ((hi == m_hi) & (lo < m_lo));
                m_hi = lower ? hi : m_hi;
                m_lo = lower ? lo : m_lo;
                m_word = lower ? word : m_word;
            };
#pragma unroll
            for (uint32_t k = 0; k < 4; ++k) {
                const bool near = tot[k] < ur, good = first[k] >= dr, step = (first[k] != 0u) & (tot[k] != 0xFFFFFFFFu);
                // {case, 2 bits; upper 30 bits of the latency}, {its lower 2 bits; accuracy from above, 16 bits; place in the line}
                const uint32_t t = near ? 0u : tot[k];
                const uint32_t hi = (near ? 0u : good ? 1u << 30 : 2u << 30) | (t >> 2);
                const uint32_t lo = (t << 30) | ((0xFFFFu - (good & !near ? 0u : first[k] >> keys)) << 8) | (4u * sub + k);
                if (step) take(hi, lo, first[k]);
            }
#pragma unroll
            for (int o = 0; o < 2; ++o) {   // the lowest of the four lanes
                auto other = [&](uint32_t v) __attribute__((always_inline)) {
                    return o == 0 ? (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xF, 0xF, true) : (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x4E, 0xF, 0xF, true);
                };
                const uint32_t o_hi = other(m_hi), o_lo = other(m_lo), o_word = other(m_word);
                take(o_hi, o_lo, o_word);
            }
            const uint32_t follows = of_quad<3>(__builtin_amdgcn_alignbit(~0u, w1.w, shift));   // (of the last lane)
            const uint32_t f_hi = packed.back(m_hi), f_lo = packed.back(m_lo), f_word = packed.back(m_word), f_next = packed.back(follows);
            const bool my = packed.mine(r0);
            r_hi = my ? f_hi : r_hi;
            r_lo = my ? f_lo : r_lo;
            r_word = my ? f_word : r_word;
            r_next = my ? f_next : r_next;
        }
        // (the lines before come first: places count from 0 in each)
        const uint32_t r_cmp = r_lo >> 8, b_cmp = b_lo >> 8;
        const bool lower = line_open(next) & ((r_hi < b_hi) | ((r_hi == b_hi) & (r_cmp < b_cmp)));
        b_hi = lower ? r_hi : b_hi;
        b_lo = lower ? r_lo : b_lo;
        b_word = lower ? r_word : b_word;
        next = line_open(next) ? r_next : next;
    }
    how = HowFar{3, 0, 0};
    if (next == kCodeRank) return kCodeRank;
    if (b_word == 0u) return kCodeNone;
    const uint32_t which = b_hi >> 30;
    const int64_t tot = ((int64_t)(b_hi & 0x3FFFFFFFu) << 2) | (int64_t)(b_lo >> 30);
    how.missed = which == 2u ? 2 : 1;
    how.over = which == 0u ? 0 : tot - (int64_t)slo;
    how.shortf = which == 1u ? 0 : (int64_t)min_acc - ((int64_t)(b_word >> keys) + (int64_t)acc_base_m1);
    return b_word & row_mask;
}

// Accuracy bound in key space: keys are acc - acc_base + 1 >= 1, so the bound is
// min_acc - acc_base + 1 limited to [1, 65536] (65536 is above every key).
__device__ __forceinline__ uint32_t acc_threshold(int32_t min_acc, int32_t acc_base_m1)
{
    const int32_t d = __builtin_elementwise_sub_sat(min_acc, acc_base_m1);   // acc_base_m1 = acc_base - 1
    return (uint32_t)(d < 1 ? 1 : (d > 65536 ? 65536 : d));
}

// ---- closest variant (the suggestion of Section 4.1 for a query that nothing satisfies): the
// variant of the slice that is first by (requirements missed, latency overshoot, accuracy
// shortfall, rank).  It is always a step.  If some step fits the latency bound it is the most
// accurate of those; else if some step is accurate enough, the fastest of those; else the fastest
// of all, the most accurate among equally fast ones; ties go to the earlier rank throughout.

// Counts of one body: accuracy keys >= dd and latency keys <= lim (none when the bound is negative).
template <class Mem>
__device__ __forceinline__ void body_counts(const Mem &mem, int nit, uint32_t body, uint32_t re, uint32_t dd,
                                            uint32_t lim, bool lim_ok, uint32_t &pa, uint32_t &ps)
{
    const uint32_t la = body + 2u * re, lt = la + 4u * re;
    uint32_t a = body, t = la;
#pragma unroll
    for (int it = 4; it >= 0; --it) {
        if (it < nit) {
            const uint32_t ca = a + (2u << it), ct = t + (4u << it);
            const uint32_t ka = mem.ld16(ca < la ? ca : la, 2u);
            const uint32_t kt = mem.ld32(ct < lt ? ct : lt, 0u);
            a = ka >= dd ? ca : a;
            t = kt <= lim ? ct : t;
        }
    }
    pa = (a - body) >> 1;
    ps = lim_ok ? (t - la) >> 2 : 0u;
}

// Smallest p in 1..re-1 whose set (tbl = address of entry 0 of A or of S, minus 4) meets `mask`.
template <class Mem>
__device__ __forceinline__ uint32_t first_meeting(const Mem &mem, uint32_t tbl, uint32_t re, uint32_t mask)
{
    uint32_t p = 0;   // the largest p found so far whose set misses the mask (set 0 is empty)
#pragma unroll
    for (uint32_t step = 16; step; step >>= 1) {
        const uint32_t c = p + step < re - 1u ? p + step : re - 1u;
        const uint32_t set = mem.ld32(tbl + 4u * c, 4u);
        p = (p + step <= re - 1u && (set & mask) == 0u) ? p + step : p;
    }
    return p + 1u;
}

// What one body offers: the step, and the keys the bodies are compared by.
struct Offer {
    uint32_t tot, acc, step;   // latency-plus-queue key, accuracy key, step number in the body
};
// kind 1: most accurate step among those within the latency bound (ps > 0 of them);
// kind 2: fastest step among those accurate enough (pa > 0 of them);
// kind 3: fastest step of all, the most accurate of equally fast ones.  The body has >= 1 step.
template <class Mem>
__device__ __forceinline__ Offer body_offer(const Mem &mem, int nit, uint32_t body, uint32_t re, int kind,
                                            uint32_t pa, uint32_t ps)
{
    const uint32_t acc_k = body, tot_k = body + 2u * re, a_tbl = body + 6u * re, s_tbl = body + 10u * re;
    Offer o;
    if (kind == 2) {
        const uint32_t mask = mem.ld32(a_tbl + 4u * pa, 4u);
        const uint32_t p = first_meeting(mem, s_tbl, re, mask);
        o.tot = mem.ld32(tot_k + 4u * p, 0u);
        o.acc = 0u;
        o.step = (uint32_t)__builtin_ctz(mem.ld32(s_tbl + 4u * p, 4u) & mask);
        return o;
    }
    uint32_t fast = ps;   // kind 3: the steps that share the smallest latency key
    o.tot = mem.ld32(tot_k + 4u, 0u);
    if (kind == 3) {
        uint32_t unused;
        body_counts(mem, nit, body, re, 0x20000u, o.tot, true, unused, fast);
    }
    const uint32_t mask = mem.ld32(s_tbl + 4u * fast, 4u);
    const uint32_t p = first_meeting(mem, a_tbl, re, mask);
    o.acc = mem.ld16(acc_k + 2u * p, 2u);
    o.step = (uint32_t)__builtin_ctz(mem.ld32(a_tbl + 4u * p, 4u) & mask);
    return o;
}

// Closest step of a slice with one or two bodies (re1 = 0: one): the step number in the slice, or -1
// when the slice has nothing to suggest, and how far that step is from the requirements (from its keys:
// no other memory is read).  body1 follows body0 in memory.  min_acc and acc_base_m1 (= accuracy
// base - 1) turn an accuracy key back into an accuracy.
struct ClosestStep {
    int32_t step;
    HowFar how;
};
template <class Mem>
__device__ __forceinline__ ClosestStep closest_step(const Mem &mem, int nit, uint32_t body0, uint32_t re0, uint32_t re1,
                                                    uint32_t dd, int32_t slo, int32_t min_acc, int32_t acc_base_m1)
{
    const ClosestStep none{-1, HowFar{3, 0, 0}};
    if (mem.ld32(body0 + 2u * re0 + 4u, 0u) == 0xFFFFFFFFu) return none;   // first latency key is the sentinel: no steps
    const uint32_t body1 = body0 + body_bytes(re0);
    const bool lim_ok = slo >= 0;
    uint32_t pa0, ps0, pa1 = 0, ps1 = 0;
    body_counts(mem, nit, body0, re0, dd, (uint32_t)slo, lim_ok, pa0, ps0);
    if (re1) body_counts(mem, nit, body1, re1, dd, (uint32_t)slo, lim_ok, pa1, ps1);
    const int kind = (ps0 | ps1) ? 1 : ((pa0 | pa1) ? 2 : 3);
    const bool use0 = kind == 1 ? ps0 > 0 : (kind == 2 ? pa0 > 0 : true);
    const bool use1 = re1 && (kind == 1 ? ps1 > 0 : (kind == 2 ? pa1 > 0 : true));
    Offer o0{0, 0, 0}, o1{0, 0, 0};
    if (use0) o0 = body_offer(mem, nit, body0, re0, kind, pa0, ps0);
    if (use1) o1 = body_offer(mem, nit, body1, re1, kind, pa1, ps1);
    bool second = use1 && !use0;
    if (use0 && use1) {   // ties go to the first body, whose steps rank earlier
        if (kind == 1) second = o1.acc > o0.acc;
        else if (kind == 2) second = o1.tot < o0.tot;
        else second = o1.tot < o0.tot || (o1.tot == o0.tot && o1.acc > o0.acc);
    }
    // A table that serves one state keeps the variants of the other states as entries nothing selects
    // (lowest accuracy key, latency key all ones).  Such an entry can be a step, and it is the closest one
    // exactly when the slice has no variant of the table's state: then there is nothing to suggest.  (Of
    // kind 1 the step is within the latency bound, so it is never such an entry.)
    const Offer o = second ? o1 : o0;
    if (kind != 1 && o.tot == 0xFFFFFFFFu) return none;
    // kind 1: within the latency bound, not accurate enough; 2: accurate enough, too slow; 3: neither
    ClosestStep c;
    c.step = second ? (int32_t)(kBodySteps + o.step) : (int32_t)o.step;
    c.how.missed = kind == 3 ? 2 : 1;
    c.how.over = kind == 1 ? 0 : (int64_t)o.tot - (int64_t)slo;
    c.how.shortf = kind == 2 ? 0 : (int64_t)min_acc - ((int64_t)o.acc + (int64_t)acc_base_m1);
    return c;
}


// ---------------------------------------------------------------- workers

__device__ __forceinline__ uint64_t lower(uint64_t a, uint64_t b) { return b < a ? b : a; }
// The instance with the smallest of these serves: by (load, worker).
__device__ __forceinline__ uint64_t instance_key(const WorkerView &wv, int32_t i)
{
    return ((uint64_t)(uint32_t)wv.inst_load[i] << 32) | (uint32_t)wv.inst_worker[i];
}

// By a whole workgroup: the worker of class c with the smallest (utilisation, number).
template <int kThreads>
__device__ __forceinline__ void best_of_class(const WorkerView &wv, int32_t c)
{
    __shared__ uint64_t s_best[kThreads / 64];
    const int32_t lo = wv.cls_off[c], hi = wv.cls_off[c + 1];
    uint64_t best = ~0ull;
    for (int32_t i = lo + (int32_t)threadIdx.x; i < hi; i += kThreads) {
        const int32_t w = wv.cls_worker[i];
        best = lower(best, ((uint64_t)(uint32_t)wv.util[w] << 32) | (uint32_t)w);   // utilisation is never negative
    }
#pragma unroll
    for (int off = 32; off; off >>= 1) best = lower(best, __shfl_xor(best, off));
    if ((threadIdx.x & 63) == 0) s_best[threadIdx.x >> 6] = best;
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int k = 1; k < kThreads / 64; ++k) best = lower(best, s_best[k]);
        wv.best_cls[c] = hi > lo ? (int32_t)(uint32_t)best : -1;
    }
}

}  // namespace
}  // namespace infaas
