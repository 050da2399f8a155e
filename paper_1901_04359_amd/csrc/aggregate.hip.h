// The aggregation that Top-k S-SGD uses (Algorithm 1, procedure TopKAllReduce), as a
// comparison workload for the tree: the P workers' k-sets are summed into one dense
// vector in rank order and averaged.  With all sets already on one GPU the AllGather of the
// procedure is a no-op; what remains is the scatter-add loop and the division by P.
#pragma once
#include "common.hip.h"

namespace gtopk {

constexpr int kAggRange = 8192;        // dense elements per range of the bounds = per block of k_scatter_mean (in LDS)
constexpr int kAggMaxP = 1024;         // workers, at most

constexpr int kAggRangeLog2 = 13;
static_assert((1 << kAggRangeLog2) == kAggRange, "range size");

constexpr int kFewP = 32;              // k_scatter_mean_few: one bit of a word per worker
constexpr int kFewRange = 2048;        // its dense elements per block: a quarter of a range of the bounds
constexpr int kFewBlock = 256;
static_assert(kAggRange % kFewRange == 0, "a block's elements lie in one range");

// bounds[g][b] = number of entries of worker g's (index-ascending) k-set with index below
// b * kAggRange, for b = 0 .. nranges: the slices that k_scatter_mean's blocks take, and between which
// k_scatter_mean_few's search on.  One binary search per bound; the searches of neighbouring bounds
// share their first probes.
__global__ __launch_bounds__(kBlock) void k_slice_bounds(
        const uint32_t* __restrict__ loc_idx, uint32_t k, uint32_t nranges,
        uint32_t* __restrict__ bounds) {
    const uint32_t b = blockIdx.x * kBlock + threadIdx.x;
    const int g = blockIdx.y;
    if (b > nranges) return;
    const uint32_t* ig = loc_idx + (size_t)g * k;
    const uint64_t target = (uint64_t)b << kAggRangeLog2;
    uint32_t lo = 0, hi = k;
    while (lo < hi) {
        const uint32_t mid = (lo + hi) >> 1;
        if ((uint64_t)ig[mid] < target) lo = mid + 1; else hi = mid;
    }
    bounds[(size_t)g * (nranges + 1) + b] = lo;
}

// Block b owns the dense elements [b*R, (b+1)*R), R = kAggRange, and keeps them in LDS.
// It reads, for every worker, the slice of that worker's k-set that falls into its range
// and lays the slices end to end ("flat" order: by worker, then by index).  Threads take
// the flat entries 1024 at a time, four each, in registers.  At one index the adds must
// happen in worker order, each one fp32 add, the first onto +0.0; entries at different
// indices are independent.  So the entries of a batch are applied in rounds: every
// pending entry bids for its index with its flat position (LDS atomic minimum), the
// winners add their value and retire, until nothing is pending.  A round retires, for
// every index, the pending entry of the lowest worker; the number of rounds is the largest
// number of workers that share one index within the batch (1 to 3 for sparse sets).
// Batches follow each other in flat order, so the order holds across batches as well.
// The range is written out once, divided by P.
__global__ __launch_bounds__(kBlock) void k_scatter_mean(
        const uint32_t* __restrict__ loc_idx, const float* __restrict__ loc_val, uint32_t P,
        uint32_t k, uint32_t m, const uint32_t* __restrict__ bounds, uint32_t nranges,
        float divisor, float* __restrict__ dense) {
    constexpr int kEpt = 4;
    constexpr uint32_t kNoBid = 0xFFFFFFFFu;
    __shared__ __align__(16) float acc[kAggRange];
    __shared__ uint32_t bid[kAggRange];
    __shared__ uint32_t s_lo[kAggMaxP];            // first entry of worker g inside the range
    __shared__ uint32_t s_off[kAggMaxP + 1];       // entries of workers < g inside the range
    __shared__ uint32_t s_wave[kBlock / kWave];
    const uint32_t t = threadIdx.x;
    const uint32_t base = blockIdx.x * (uint32_t)kAggRange;          // < m by the launch grid
    const uint32_t span = m - base < (uint32_t)kAggRange ? m - base : (uint32_t)kAggRange;
    for (uint32_t g = t; g < P; g += kBlock) {
        const uint32_t* bg = bounds + (size_t)g * (nranges + 1) + blockIdx.x;
        uint32_t lo = bg[0], hi = bg[1];
        // always lo <= hi <= k for a sorted set; keeps every access in bounds for any other
        if (hi > k) hi = k;
        if (lo > hi) lo = hi;
        s_lo[g] = lo;
        s_off[g + 1] = hi;                         // holds the end for now
    }
    for (uint32_t i = t; i < (uint32_t)kAggRange; i += kBlock) { acc[i] = 0.0f; bid[i] = kNoBid; }
    __syncthreads();
    // counts -> exclusive offsets (up to 4 workers per thread)
    {
        constexpr int kPer = kAggMaxP / kBlock;
        uint32_t c[kPer], sum = 0;
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            const uint32_t g = t * kPer + j;
            c[j] = g < P ? s_off[g + 1] - s_lo[g] : 0u;
            sum += c[j];
        }
        __syncthreads();                  // every end has been read before offsets overwrite them
        uint32_t total;
        uint32_t run = block_incl_scan(sum, s_wave, total) - sum;
        if (t == 0) s_off[0] = 0u;
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            const uint32_t g = t * kPer + j;
            run += c[j];
            if (g < P) s_off[g + 1] = run;
        }
    }
    __syncthreads();
    const uint32_t total = s_off[P];
    // worker that holds flat entry e: the last g with s_off[g] <= e (empty workers skipped)
    auto worker_of = [&](uint32_t e) {
        uint32_t lo = 0, hi = P;          // answer in [lo, hi)
        while (hi - lo > 1) {
            const uint32_t mid = (lo + hi) >> 1;
            if (s_off[mid] <= e) lo = mid; else hi = mid;
        }
        return lo;
    };
    for (uint32_t c0 = 0; c0 < total; c0 += kBlock * kEpt) {
        // thread t takes the flat entries c0 + 4t .. c0 + 4t + 3: its bids order them
        uint32_t ei[kEpt];
        float ev[kEpt];
        bool pending[kEpt];
#pragma unroll
        for (int u = 0; u < kEpt; ++u) {
            const uint32_t e = c0 + t * kEpt + u;
            pending[u] = e < total;
            ei[u] = 0;
            ev[u] = 0.0f;
            if (pending[u]) {
                const uint32_t g = worker_of(e);
                const size_t j = (size_t)g * k + s_lo[g] + (e - s_off[g]);
                ei[u] = loc_idx[j] - base;
                ev[u] = loc_val[j];
                pending[u] = ei[u] < (uint32_t)kAggRange;      // always true for sorted sets
            }
        }
        bool any = true;
        while (any) {                     // block-uniform: `any` comes from a block-wide vote
#pragma unroll
            for (int u = 0; u < kEpt; ++u)
                if (pending[u]) atomicMin(&bid[ei[u]], t * kEpt + u);
            __syncthreads();
            bool win[kEpt];
#pragma unroll
            for (int u = 0; u < kEpt; ++u) win[u] = pending[u] && bid[ei[u]] == t * kEpt + u;
            __syncthreads();
            bool left = false;
#pragma unroll
            for (int u = 0; u < kEpt; ++u) {
                if (win[u]) {
                    acc[ei[u]] = acc[ei[u]] + ev[u];
                    bid[ei[u]] = kNoBid;
                    pending[u] = false;
                }
                left = left || pending[u];
            }
            any = __syncthreads_or(left) != 0;
        }
    }
    __syncthreads();
    float* out = dense + base;                      // 16-byte aligned: base is a multiple of kAggRange
    if (span == (uint32_t)kAggRange) {
        for (uint32_t i = 4 * t; i < (uint32_t)kAggRange; i += 4 * kBlock) {
            const float4 a = *reinterpret_cast<const float4*>(&acc[i]);
            *reinterpret_cast<float4*>(out + i) =
                make_float4(a.x / divisor, a.y / divisor, a.z / divisor, a.w / divisor);
        }
    } else {
        for (uint32_t i = t; i < span; i += kBlock) out[i] = acc[i] / divisor;
    }
}

// The same for at most 32 workers.  What bounded k_scatter_mean was latency: with a bid per
// element its 74 KB of LDS leave two blocks of four waves per CU, and every round of bids costs
// three barriers.  Here a block owns kFewRange elements (17 KB) and, instead of a bid, keeps per
// element the set of workers of the batch that hold it, one bit each: an entry's turn is the number
// of lower workers in that set, so turns need one barrier each and no vote.  The workers' entries crowd
// into a few ranges (the layers with large gradients), and the blocks of those take as long as the
// launch: a quarter of a range per block shortens them, and each finds its part of every worker's
// entries by two searches inside the range's bounds.  The average of 32 workers at m = 25,557,032 in us,
// k_scatter_mean / blocks of 4096 that read the whole range / 2048 / 1024 elements:
//   k = 25,557  103 / 63 / 50 / 50     k = 255,570  291 / 174 / 135 / 122     the same in one layer  131 / 80 / 76 / 108
// and at m = 61,100,840, k = 61,101 (many empty ranges)  89 / 52 / 51 / 74.
__global__ __launch_bounds__(kFewBlock) void k_scatter_mean_few(
        const uint32_t* __restrict__ loc_idx, const float* __restrict__ loc_val, uint32_t P,
        uint32_t k, uint32_t m, const uint32_t* __restrict__ bounds, uint32_t nranges,
        float divisor, float* __restrict__ dense) {
    constexpr int kEpt = 4;
    constexpr uint32_t kParts = kAggRange / kFewRange;
    __shared__ __align__(16) float acc[kFewRange];
    __shared__ __align__(16) uint32_t who[kFewRange];      // workers of the batch that hold the element
    __shared__ uint32_t s_lo[kFewP];                       // first entry of worker g inside the range
    __shared__ uint32_t s_off[kFewP + 1];                  // entries of workers < g inside the range
    __shared__ uint32_t s_last;                            // last turn of the batch
    const uint32_t t = threadIdx.x;
    const uint32_t range = blockIdx.x / kParts;
    const uint32_t base = range * (uint32_t)kAggRange + (blockIdx.x % kParts) * (uint32_t)kFewRange;
    if (base >= m) return;                                 // block-uniform
    const uint32_t span = m - base < (uint32_t)kFewRange ? m - base : (uint32_t)kFewRange;
    if (t < (uint32_t)kWave) {
        // lane g: where the block's part of worker g's entries in the range starts; lane 32 + g: where it ends
        const uint32_t g = t % (uint32_t)kFewP;
        uint32_t lo = 0, hi = 0;
        if (g < P) {
            const uint32_t* bg = bounds + (size_t)g * (nranges + 1) + range;
            lo = bg[0];
            hi = bg[1];
            // always lo <= hi <= k for a sorted set; keeps every access in bounds for any other
            if (hi > k) hi = k;
            if (lo > hi) lo = hi;
            const uint32_t first = t < (uint32_t)kFewP ? base : base + (uint32_t)kFewRange;
            const uint32_t* set = loc_idx + (size_t)g * k;
            while (lo < hi) {
                const uint32_t mid = (lo + hi) >> 1;
                if (set[mid] < first) lo = mid + 1; else hi = mid;
            }
        }
        hi = (uint32_t)__shfl_xor((int)lo, kFewP);
        if (t >= (uint32_t)kFewP || hi < lo) hi = lo;      // (hi < lo: not a sorted set)
        const uint32_t incl = wave_incl_scan(hi - lo);
        if (t < P) {
            s_lo[t] = lo;
            s_off[t + 1] = incl;
        }
        if (t == 0) { s_off[0] = 0u; s_last = 0u; }
    }
    for (uint32_t i = 4 * t; i < (uint32_t)kFewRange; i += 4 * kFewBlock) {
        *reinterpret_cast<float4*>(&acc[i]) = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        *reinterpret_cast<uint4*>(&who[i]) = make_uint4(0u, 0u, 0u, 0u);
    }
    __syncthreads();
    const uint32_t total = s_off[P];
    if (total == 0u) {                                     // nobody holds anything here (block-uniform)
        for (uint32_t i = 4 * t; i < span; i += 4 * kFewBlock) {
            if (i + 4 <= span) *reinterpret_cast<float4*>(dense + base + i) = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            else for (uint32_t j = i; j < span; ++j) dense[base + j] = 0.0f;
        }
        return;
    }
    for (uint32_t c0 = 0; c0 < total; c0 += kFewBlock * kEpt) {
        uint32_t ei[kEpt], eg[kEpt];
        float ev[kEpt];
        bool mine[kEpt];
#pragma unroll
        for (int u = 0; u < kEpt; ++u) {
            const uint32_t e = c0 + u * kFewBlock + t;
            mine[u] = e < total;
            ei[u] = 0; eg[u] = 0; ev[u] = 0.0f;
            if (mine[u]) {
                uint32_t lo = 0, hi = P;                   // the last g with s_off[g] <= e
                while (hi - lo > 1) {
                    const uint32_t mid = (lo + hi) >> 1;
                    if (s_off[mid] <= e) lo = mid; else hi = mid;
                }
                const size_t j = (size_t)lo * k + s_lo[lo] + (e - s_off[lo]);
                eg[u] = lo;
                ei[u] = loc_idx[j] - base;
                ev[u] = loc_val[j];
            }
        }
#pragma unroll
        for (int u = 0; u < kEpt; ++u) {
            mine[u] = mine[u] && ei[u] < (uint32_t)kFewRange;      // always for a sorted set; stays in LDS for any other
            if (mine[u]) atomicOr(&who[ei[u]], 1u << eg[u]);
        }
        __syncthreads();
        uint32_t turn[kEpt], last = 0;
#pragma unroll
        for (int u = 0; u < kEpt; ++u) {
            turn[u] = mine[u] ? (uint32_t)__popc(who[ei[u]] & ((1u << eg[u]) - 1u)) : 0u;
            last = turn[u] > last ? turn[u] : last;
        }
        if (last) atomicMax(&s_last, last);
        __syncthreads();
        last = s_last;
        for (uint32_t r = 0; r <= last; ++r) {             // block-uniform
            if (r) __syncthreads();
#pragma unroll
            for (int u = 0; u < kEpt; ++u)
                if (mine[u] && turn[u] == r) acc[ei[u]] = acc[ei[u]] + ev[u];
        }
        // (every turn has been worked out before the barrier above: the sets can be cleared)
#pragma unroll
        for (int u = 0; u < kEpt; ++u)
            if (mine[u]) who[ei[u]] = 0u;
        __syncthreads();
        if (t == 0) s_last = 0u;                           // read by all, set again behind a barrier
    }
    float* out = dense + base;                             // 16-byte aligned: base is a multiple of kFewRange
    if (span == (uint32_t)kFewRange) {
        for (uint32_t i = 4 * t; i < (uint32_t)kFewRange; i += 4 * kFewBlock) {
            const float4 a = *reinterpret_cast<const float4*>(&acc[i]);
            *reinterpret_cast<float4*>(out + i) =
                make_float4(a.x / divisor, a.y / divisor, a.z / divisor, a.w / divisor);
        }
    } else {
        for (uint32_t i = t; i < span; i += kFewBlock) out[i] = acc[i] / divisor;
    }
}

}  // namespace gtopk
