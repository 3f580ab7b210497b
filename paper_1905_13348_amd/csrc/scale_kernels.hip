// Scaling decision on a change in query load (Section 4.2.2, scaling up): for a running variant,
// its instance count and the incoming load, either nothing, or replicate the variant, or upgrade
// to a variant of the same model architecture with a higher saturation throughput that meets the
// latency objective -- whichever is cheaper by the cost function of the integer program of
// Section 4.2.1, C * (delta + lambda * T_load * max(delta, 0)) summed over the touched variants.
//
// One lane per request, one cache line per request.  Per batch size and architecture the host keeps
// the candidates for an upgrade sorted by descending throughput and without the variants that can
// never win: v loses to w for every request when w has at least v's throughput, at most v's latency
// and a lower cost per instance (or the same and a lower row), because w then passes every test v
// passes and needs no more instances.  The candidates of a running variant are the prefix of that
// list with a higher throughput than its own; the first five of them are copied, with everything
// else the decision reads about the variant, into a 128-byte block per (batch size, variant), so a
// request costs one uncoalesced line (longer prefixes continue in the shared list).  All costs are
// exact integers (times 1,000,000, because lambda is per second and the loading latency in
// microseconds) of at most 94 bits.
//
// Scaling down (Section 4.2.2, second algorithm) is the same kernel on a second set of blocks: keep,
// or remove one instance when the others still carry the load, or downgrade to a variant of the same
// architecture with a lower hardware cost that meets the latency objective -- whichever lowers the
// same objective most.  There the lists are sorted by ascending hardware cost, the candidates of a
// running variant are the prefix with a lower one, and v loses to w for every request when w
// besides has at most v's hardware cost.
#include "internal.h"

namespace infaas {

namespace {

constexpr int kThreads = 64;   // one wavefront
constexpr int kChunk = 2;   // candidates of a list read together

// An exact cost of up to 94 bits, and below its last word who it belongs to: 0 for the running variant, the caller row + 1 for a
// switch.  So the lower of two is the lower cost, and at a tie the running variant, else the lower row.
struct Offer {
    uint64_t high;
    uint32_t low, who;
};
__device__ __forceinline__ bool operator<(const Offer &a, const Offer &b)
{
    const uint64_t x = ((uint64_t)a.low << 32) | a.who, y = ((uint64_t)b.low << 32) | b.who;
    return (a.high < b.high) | ((a.high == b.high) & (x < y));
}
// n instances at `unit` each (below 2^62)
__device__ __forceinline__ Offer offer_of(uint64_t unit, uint32_t n, uint32_t who)
{
    const uint64_t lo = (uint64_t)(uint32_t)unit * n;
    return Offer{(unit >> 32) * n + (lo >> 32), (uint32_t)lo, who};
}

// ceil(need / per) for need < 2^31 and 1 <= per < 2^31: the hardware's estimate of 1 / per (v_rcp_f64, good to 2^-20 and
// better) after one Newton step is within 2^-39 of it, relatively, so the quotient's integer part is the exact floor or one
// beside it, and the remainder (which fits 32 bits in all three cases) tells which.
__device__ __forceinline__ uint32_t ceil_div(uint32_t need, uint32_t per)
{
    const double d = (double)per, r = __builtin_amdgcn_rcp(d);
    const double inv = __builtin_fma(__builtin_fma(-d, r, 1.0), r, r);
    const uint32_t q = (uint32_t)((double)need * inv);
    const int32_t rest = (int32_t)(need - q * per);
    return q + (uint32_t)(rest > 0) + (uint32_t)(rest > (int32_t)per);
}

// The loads in front of this are issued together and arrive together: without it the compiler moves each of a block's words
// behind the branch that first needs it, and a request waits for memory several times.
__device__ __forceinline__ void arrived(uint4 &v) { asm volatile("" : "+v"(v.x), "+v"(v.y), "+v"(v.z), "+v"(v.w)); }

// Bound by the requests' lines: 4M of them on 102 MB of blocks, read by a kernel that does nothing else, take 86 us together with
// the fields and results, this kernel 99; the continuations of long lists, 0.2 lines per request more, come from L2 (whole lists
// instead of their ends: 99.8).  Candidates are computed for every lane and masked, without branches; 32-bit quotients (the need is rounded up
// to whole queries per second once: ceil(ceil(x / 100) / q) = ceil(x / (100 q))) and 96-bit costs.
template <bool kDown>
__global__ __launch_bounds__(kThreads) void k_scale(ScaleView sv, int64_t R, const int32_t *__restrict__ r_variant,
                                                    const int32_t *__restrict__ r_instances,
                                                    const int32_t *__restrict__ r_load_qps,
                                                    const int32_t *__restrict__ r_slo_us,
                                                    const int32_t *__restrict__ r_batch_idx,
                                                    int32_t *__restrict__ out_action, int32_t *__restrict__ out_variant,
                                                    int32_t *__restrict__ out_instances)
{
    for (int64_t r0 = (int64_t)blockIdx.x * kThreads; r0 < R; r0 += (int64_t)gridDim.x * kThreads) {
        const int64_t r = r0 + threadIdx.x;
        const bool in = r < R;
        const int64_t at = in ? r : r0;
        const int32_t cur = __builtin_nontemporal_load(r_variant + at);
        const int32_t b = __builtin_nontemporal_load(r_batch_idx + at);
        const int32_t n_cur = __builtin_nontemporal_load(r_instances + at);
        const int32_t load = __builtin_nontemporal_load(r_load_qps + at);
        const int32_t slo = __builtin_nontemporal_load(r_slo_us + at);
        const bool valid = (uint32_t)cur < (uint32_t)sv.V && (uint32_t)b < (uint32_t)sv.B &&
                           (uint32_t)n_cur <= 1000000u && (uint32_t)load <= 1000000000u;
        // the request's block: one cache line, all of it requested at once
        const uint4 *blk = (const uint4 *)((kDown ? sv.blocks_down : sv.blocks) + ((int64_t)(valid ? b : 0) * sv.V + (valid ? cur : 0)) * kScaleBlockWords);
        uint4 head = blk[0];      // {throughput, hardware cost, cost of one instance}
        uint4 more = blk[1];      // {latency, candidates, their list, row of the fifth}
        uint4 slot[kScaleInBlock];
#pragma unroll
        for (int j = 0; j < kScaleInBlock; ++j) slot[j] = blk[2 + j];   // {throughput, latency, cost of one instance}
        uint4 rows4 = blk[7];
        arrived(head);
        arrived(more);
#pragma unroll
        for (int j = 0; j < kScaleInBlock; ++j) arrived(slot[j]);
        arrived(rows4);
        const uint32_t slot_row[kScaleInBlock] = {rows4.x, rows4.y, rows4.z, rows4.w, more.w};
        const uint32_t own_qps = head.x;
        const uint64_t own_unit = ((uint64_t)head.w << 32) | head.z;
        // whole queries per second the instances have to carry (for valid requests at most 2 * 10^9)
        const uint32_t need = (uint32_t)(((uint64_t)(uint32_t)load * (uint32_t)sv.slack_pct + 99u) / 100u);
        // everything is compared with the credit for unloading the running instances added, so
        // that no difference can become negative
        const uint64_t saved = (uint64_t)head.y * (uint32_t)n_cur * 1000000u;   // < 2^61
        const bool scaling = valid && (kDown || (uint64_t)own_qps * (uint32_t)n_cur < need);
        const int32_t m = scaling ? (int32_t)more.y : 0;
        Offer best{~0ull, 0u, 0u};   // (no cost comes near)
        uint32_t best_n = 0;
        bool remove = false;
        if constexpr (!kDown) {   // replicate
            const uint32_t n = ceil_div(need, own_qps) - (uint32_t)n_cur;
            Offer o = offer_of(own_unit, n, 0u);
            const uint64_t low = (uint64_t)o.low + (uint32_t)saved;
            o.high += (saved >> 32) + (low >> 32);
            o.low = (uint32_t)low;
            if ((int32_t)more.x <= slo) { best = o; best_n = n; }
        } else {
            // keeping everything costs `saved` on this scale; removing one instance one hardware cost
            // less, allowed when at least one instance stays and the rest carries the load
            remove = n_cur >= 2 && (uint64_t)own_qps * (uint32_t)(n_cur - 1) >= need && head.y > 0u;   // (at no hardware cost there is nothing to gain)
            const uint64_t cost = remove ? saved - (uint64_t)head.y * 1000000u : saved;
            best = Offer{cost >> 32, (uint32_t)cost, 0u};
        }
        // a switch to a candidate (which has a higher throughput, resp. a lower hardware cost, than cur
        // by construction); at least one instance serves after a downgrade
        auto offer = [&](bool on, uint32_t qps, int32_t lat, uint64_t unit, uint32_t row) __attribute__((always_inline)) {
            uint32_t n = ceil_div(need, qps);
            if (kDown) n = n < 1u ? 1u : n;
            const Offer o = offer_of(unit, n, row + 1u);
            const bool better = on & (lat <= slo) & (o < best);
            if (better) { best = o; best_n = n; }
        };
        // the rest of a longer prefix, from the shared list, two at a time; requested before the block's own are looked at
        const ScaleCand *all = kDown ? sv.cand_down : sv.cand;
        const int32_t rest = m - kScaleInBlock;
        uint4 cand[kChunk];
        uint32_t cand_row[kChunk];
        // Only lanes with something left read: where lists are long most have nothing, and a read of some line that is there anyway
        // costs them as much as their own did (architectures of 400 variants of which nothing beats another, 4M requests: 2480 us so, 2024
        // masked; of 100, 710 and 624; of 12 random ones, 82.7 and 81.8).
        auto request = [&](int32_t i0) __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < kChunk; ++j) {
                cand[j] = make_uint4(1u, 0u, 0u, 0u);   // (a throughput of 1)
                cand_row[j] = 0u;
                if (i0 + j < rest) {
                    const ScaleCand *c = all + (int64_t)more.z + i0 + j;
                    cand[j] = *(const uint4 *)c;
                    cand_row[j] = (uint32_t)c->row;
                }
            }
        };
        int32_t i0 = 0;
        bool longer = __ballot(rest > 0) != 0ull;
        if (longer) request(0);
#pragma unroll
        for (int j = 0; j < kScaleInBlock; ++j)
            offer(j < m, slot[j].x, (int32_t)slot[j].y, ((uint64_t)slot[j].w << 32) | slot[j].z, slot_row[j]);
        while (longer) {
#pragma unroll
            for (int j = 0; j < kChunk; ++j) {
                arrived(cand[j]);
                offer(i0 + j < rest, cand[j].x, (int32_t)cand[j].y, ((uint64_t)cand[j].w << 32) | cand[j].z, cand_row[j]);
            }
            i0 += kChunk;
            longer = __ballot(rest > i0) != 0ull;
            if (longer) request(i0);
        }
        int32_t action = 0, variant = -1, instances = 0;
        if (kDown ? best.who != 0u : best.high != ~0ull) {
            action = best.who ? 2 : 1;
            variant = best.who ? (int32_t)best.who - 1 : cur;
            instances = (int32_t)best_n;
        } else if (kDown ? remove : true) {
            action = kDown ? 1 : 3;
            variant = kDown ? cur : -1;
            instances = kDown ? 1 : 0;
        }
        if (!scaling) { action = 0; variant = -1; instances = 0; }
        if (in) {
            __builtin_nontemporal_store(action, out_action + r);
            __builtin_nontemporal_store(variant, out_variant + r);
            __builtin_nontemporal_store(instances, out_instances + r);
        }
    }
}

}  // namespace

hipError_t launch_scale(const ScaleView &sv, bool down, int64_t R, const int32_t *r_variant, const int32_t *r_instances,
                        const int32_t *r_load_qps, const int32_t *r_slo_us, const int32_t *r_batch_idx,
                        int32_t *out_action, int32_t *out_variant, int32_t *out_instances, int num_cus,
                        hipStream_t st, const LaunchEvents *ev)
{
    if (R <= 0) return hipSuccess;
    const int64_t want = (R + kThreads - 1) / kThreads;
    // one request per lane (to 2^26 of them): the loop over a smaller grid makes every lane wait for its request's line
    // before it asks for the next one's fields (4M requests 3% longer with 32 workgroups per compute unit).  One wavefront to a
    // workgroup, so that none waits for its neighbours to leave, and lists two candidates at a time: us for 4M / 700,001 requests
    // 99 / 21.1, with four at a time and four wavefronts 101.0 / 22.2; with a compiler that moved every word's load behind its
    // first use, and branches, 128-bit quotients and costs 125.8 / 23.9.
    const int64_t blocks = want < (int64_t)num_cus * 4096 ? want : (int64_t)num_cus * 4096;
    if (down)
        return launch_kernel(ev, k_scale<true>, dim3((unsigned)blocks), dim3(kThreads), 0, st, sv, R, r_variant,
                             r_instances, r_load_qps, r_slo_us, r_batch_idx, out_action, out_variant, out_instances);
    return launch_kernel(ev, k_scale<false>, dim3((unsigned)blocks), dim3(kThreads), 0, st, sv, R, r_variant, r_instances,
                         r_load_qps, r_slo_us, r_batch_idx, out_action, out_variant, out_instances);
}

}  // namespace infaas
