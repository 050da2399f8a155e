// The step at large densities (several percent of the row): everything behind the streaming pass works on
// index groups - group g of any set holds its entries with indices [g * kGroup, (g + 1) * kGroup) - and on a
// two-sided speculative bracket of the k-th key instead of a lower bound alone.
//
// At these densities the candidates of a worker are millions of entries that lie close together: writing
// them out in the pass, walking them and reading them again costs more than reading the parts of the row that
// hold them once more.  So a producer (the pass; the union of a pair) keeps nothing but, per group, the number
// of keys above the bracket and the keys inside it (a tenth of k), histogrammed:
//   k_group_pass    acc = residual + grad, written back; per group the count of keys >= hi, the keys in
//                   [lo, hi), and which stretches of 256 elements hold any key >= lo
//   k_group_walk    the bin of the k-th key from the histogram of the bracket's keys; per group the count of
//                   keys above that bin, the keys inside it into a short list.  One block per pair of the next
//                   round picks that round's bracket from a sample of the pair's union.
//   k_group_finish  the exact k-th key and ties, output position of every group (one block per set)
//   k_group_select  two workers' rows are read again, group by group: their selected entries are emitted in
//                   index order, and their union, formed in registers, is counted for the first round
//   k_group_merge   the same for the rounds behind it: the pair's union is formed in LDS, by index, from the
//                   sub-lists of its two operands, selected and emitted; two such results side by side are the
//                   next round's union, which is counted before it leaves the registers
//   k_group_restore residual slots whose index is in the worker's set and in the global one become +0.0
// A step at m = 25,557,032, P = 32, k = 6,389,258 (54 layers) in us, lists of candidates and merged sets / this: 6578 / 4700
// (pass 2122 / 1700, local select and first union 1630 / 800, rounds behind it 1970 / 1350, restore 852 / 790).
// Every list is written once and read once per round, no merged set is ever stored, and no cut point is
// searched for: the sub-lists of a group are known from the groups' output positions.
// A set whose k-th key lies outside its bracket (the sample misled) is counted whole by k_group_walk and gets another
// bracket from that, whose keys several blocks of k_group_finish collect.  A step whose rows all mislead the sampler, of 24
// layers, in us (lists / this; with one block of k_group_finish that reads all keys 6200 at the third of these sizes, 55,500 and
// 67,800 at the first two):
//   m = 25.6 M  P = 4   k = m/4   2260 .. 2890 / 1760      m = 25.6 M  P = 32  k = m/4     15,000 .. 18,600 / 9600
//   m = 4.2 M   P = 4   k = m/8     390 .. 475 / 530       m = 4.2 M   P = 2   k = 0.31 m       277 .. 315 / 467
// So short rows lose to the lists there: without such rows the last two take 221 / 206 and 186 / 145.  (The walk reads its
// keys with sixteen loads in flight per lane; as long as each was changed inside its own condition, one after the other, the
// walk of two rows of 4.2 M took 147 us instead of 49.)
#pragma once
#include "common.hip.h"

namespace gtopk {

constexpr int kGrpWaves = 8;                            // waves per block of the select and the merge
constexpr int kGrpBlock = kGrpWaves * kWave;            // threads
constexpr int kGrpPer = 16;                             // elements per thread: 64 consecutive ones per wave and step
constexpr uint32_t kGroup = kGrpBlock * kGrpPer;        // indices per group
constexpr uint32_t kGroupLog2 = 13;
static_assert(kGroup == 1u << kGroupLog2, "a group is a block's");
constexpr uint32_t kMaxIndexGroups = 8192;              // groups per row, at most
constexpr uint32_t kAbsent = 0xFFFFFFFFu;               // no value
constexpr uint32_t kZeroSum = 0x80000000u;              // -0.0: the other "no value", see Plain
constexpr uint32_t kInfKey = 0x7F800000u;               // a bracket ends here at most: its ends are numbers
constexpr int kBrkBins = 2048;                          // a bracket's histogram: 1024 bins at most ..
constexpr uint32_t kAboveBin = (uint32_t)kBrkBins - 1;  // .. and the count of the keys above
constexpr uint32_t kMissed = 0xFFFFFFFFu;               // GroupSets::d1 of a set whose bracket does not hold the k-th key
constexpr uint32_t kTopBins = 2048;                     // a key's bits 30 .. 20
constexpr uint32_t kAllBins = kTopBins + 1024;          // .. and bits 19 .. 10 of the keys in the k-th key's one of those
constexpr uint32_t kPlainRun = 0xFFFFFFFFu;             // run.w: the keys are stored (else: all of them are this key)

// A value as it is kept in registers and LDS, where kAbsent stands for "none" (one NaN pattern of either sign gives way
// to its neighbour, so that no key of a value is kAbs).
__device__ __forceinline__ uint32_t present(uint32_t bits) { return (bits & kAbs) == kAbs ? bits - 1u : bits; }
__device__ __forceinline__ uint32_t present_key(uint32_t bits) { return (bits & kAbs) < kAbs - 1u ? bits & kAbs : kAbs - 1u; }
// Whether x lies in [lo, hi), one subtraction and one comparison: with hi = kAbs and x = v & kAbs also whether v is
// there at all.
__device__ __forceinline__ bool within(uint32_t x, uint32_t lo, uint32_t hi) { return x - lo < hi - lo; }

// The same uniform value, as one the compiler knows nothing of: a loop that compares a thread's elements with it a
// second time then does that, where the masks of the first time would be kept and spilled.
__device__ __forceinline__ uint32_t once_more(uint32_t x) {
    asm volatile("" : "+v"(x));
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)x);
}

// base[offset] for a uniform base: one address register and a lane's 32-bit offset
__device__ __forceinline__ void store_at(uint32_t* base, uint32_t offset, uint32_t x) {
    *reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(base) + (offset << 2)) = x;
}
__device__ __forceinline__ uint32_t load_at(const uint32_t* base, uint32_t offset) {
    return *reinterpret_cast<const uint32_t*>(reinterpret_cast<const char*>(base) + (offset << 2));
}

// Per-set state; sets are numbered through: the workers' 0 .. P-1, then the pairs of each round.
struct GroupSets {
    uint32_t* hist;      // [sets][kBrkBins] bracket keys, the last one the keys above                      } cleared
    uint32_t* hist_all;  // [sets][kAllBins] all keys of a set that missed its bracket                      } before
    uint32_t* list_cnt;  // [sets]                                                                          } a step
    uint32_t* arrived;   // [sets] blocks that have collected their groups of such a set                    }
    uint32_t* brk_cnt;   // [P] bracket keys that the pass has stored (or tried to)                         }
    uint32_t* lo;        // [sets] the bracket
    uint32_t* hi;
    uint32_t* d1;        // [sets] bin of the k-th key, or kMissed
    uint32_t* krem;      // [sets] its rank in there, from the top
    uint32_t* T;         // [sets] the k-th largest key
    uint32_t* need;      // [sets] entries with key == T to take
    uint4* run;          // [sets][ngroups] bracket keys: (first, count, keys above the bracket, kPlainRun or the one key)
    uint32_t* grp_gt;    // [sets][ngroups] keys above bin d1
    uint2* off;          // [sets][ngroups + 1] entries with key > T / == T in the groups before
    uint32_t* tail;      // [P][ngroups][3] see k_group_pass
    uint64_t* mask;      // [P][ngroups + 1] stretches of 256 elements that hold a key >= lo
    uint32_t m, ngroups;
};

// Bracket [lo, hi) of a set's k-th key, cut into 513 to 1024 bins of equal width (fewer if it is narrower than that).
struct Bracket {
    uint32_t lo, hi, shift;
    __device__ __forceinline__ Bracket(const GroupSets& gs, uint32_t id) : lo(gs.lo[id]), hi(gs.hi[id]) {
        const uint32_t bits = 32u - (uint32_t)__builtin_clz((hi > lo ? hi - lo - 1u : 0u) | 1u);
        shift = bits > 10u ? bits - 10u : 0u;
    }
    __device__ __forceinline__ bool holds(uint32_t key) const { return key - lo < hi - lo; }      // (hi >= lo)
    __device__ __forceinline__ uint32_t bin(uint32_t key) const { return (key - lo) >> shift; }
    __device__ __forceinline__ uint32_t bin_lo(uint32_t b) const { return lo + (b << shift); }
};

// Which of a group's elements stand for it in the sample of a union: of the 1024 that a wave holds, q lanes of
// one step.  Scattered by a hash (odd multipliers and xor-shifts, any that mix the low bits serve), so that no period of the
// data falls in with them.
__device__ __forceinline__ uint32_t sample_hash(uint32_t g, uint32_t wave) {
    uint32_t h = g * 0x9E3779B1u + wave * 0x85EBCA6Bu;
    h ^= h >> 15;
    h *= 0x2C1B3C6Du;
    return h ^ (h >> 13);
}
__device__ __forceinline__ uint32_t sample_step(uint32_t h) { return h & (kGrpPer - 1); }
__device__ __forceinline__ uint32_t sample_lane(uint32_t h, uint32_t l, uint32_t q) {
    return ((h >> 8) + l * (kWave / q)) & (kWave - 1);
}

// ---------------------------------------------------------------------------------
// the streaming pass
// ---------------------------------------------------------------------------------

// The block shape, the loads and the stores are k_accum_filter's.  A wave's elements follow each other, so a
// block's waves are cut evenly between its kGroupsPerBlock groups.  Vector accesses are aligned on v = index +
// head (see k_accum_filter), groups are cut by index: the first `head` elements on v of a group belong to the group
// before; their keys go to its tail[] and nowhere else (the histogram apart).
// A group crowded with bracket keys that are all equal (zeros, signs) is kept as that key and a count.
// Blocks are half as long as k_accum_filter's, and each XCD streams one eighth of all rows from end to end instead of
// every eighth chunk (at m = 25,557,032, P = 32, k = 6.4 M / 1.85 M: 1743 / 1715 us with blocks of 2^15 in the order of their
// numbers, 1719 / 1699 by XCD, 1704 / 1688 with blocks of 2^14).
// Bound by HBM as k_accum_filter is, and without its candidate lists: at m = 25,557,032, P = 32, k = 6.4 M it writes
// 0.25 GB behind the rows (3.52 GB by the counters, 3.27 the rows) where the lists took 1.9 GB.
constexpr int kGrpPassIters = 8;                        // float4 per lane and array: blocks of 2^14 elements
constexpr uint32_t kGrpPassChunk = kGrpPassIters * 4 * kSBlock;
__global__ __launch_bounds__(kSBlock) void k_group_pass(
        const float* __restrict__ grad, float* __restrict__ res, int64_t stride, GroupSets gs,
        float* __restrict__ keys, uint32_t cap, uint32_t* __restrict__ cand_count) {
    constexpr int kWaves = kSBlock / kWave, ITERS = kGrpPassIters;
    constexpr uint32_t kSpan = ITERS * 4 * kWave;            // elements per wave
    constexpr int kWavesPerGroup = (int)(kGroup / kSpan);
    constexpr int kGroupsPerBlock = kWaves / kWavesPerGroup;
    static_assert(kGroupsPerBlock >= 1, "a block holds whole groups");
    __shared__ uint32_t s_in[kWaves], s_hi[kWaves], s_mask[kWaves], s_max[kWaves], s_min[kWaves];
    __shared__ uint32_t s_base;
    __shared__ uint32_t s_h[kBrkBins];
    for (int b = threadIdx.x; b < kBrkBins; b += kSBlock) s_h[b] = 0u;      // a barrier follows
    uint32_t chunk, w;
    {
        const uint32_t id = blockIdx.y * gridDim.x + blockIdx.x, per = gridDim.x * gridDim.y / 8u;
        const uint32_t at = id < per * 8u ? (id & 7u) * per + (id >> 3) : id;
        w = at / gridDim.x;
        chunk = at - w * gridDim.x;
    }
    const uint32_t lane = lane_id();
    const uint32_t wave = threadIdx.x / kWave;
    const uint32_t head = (uint32_t)(((int64_t)w * stride) & 3);
    const float* g = grad + (int64_t)w * stride - head;
    float* r = res + (int64_t)w * stride - head;
    const uint32_t vend = head + gs.m;
    const Bracket bk(gs, w);
    const uint32_t wbase = chunk * (kSpan * (uint32_t)kWaves) + wave * kSpan;

    // Sums of the elements that this wave counts for its own group: those in the row and not among the first `head` of a
    // group.  Its keys are compared as numbers, |sum| with the bracket's ends (a NaN is above all); where elements are missing
    // (edge) as integers, which the kAbsent in their place fails.
    uint32_t a[ITERS][4];
    const uint32_t vgroup = wbase >> kGroupLog2;                 // (wave-uniform) group on v
    const bool has_tail = head && (wbase & (kGroup - 1u)) == 0u;
    const bool whole = wbase >= head && wbase + kSpan <= vend;
    const bool edge = !whole || (has_tail && bk.lo == 0u);       // wave-uniform
    if (whole) {
        floatx4 gv[ITERS], rv[ITERS];
#pragma unroll
        for (int i = 0; i < ITERS; ++i) {
            const uint32_t v = wbase + i * 256 + lane * 4;
            gv[i] = __builtin_nontemporal_load(reinterpret_cast<const floatx4*>(g + v));
            rv[i] = __builtin_nontemporal_load(reinterpret_cast<const floatx4*>(r + v));
        }
#pragma unroll
        for (int i = 0; i < ITERS; ++i) {
            const uint32_t v = wbase + i * 256 + lane * 4;
            const floatx4 s = rv[i] + gv[i];                     // four independent fp32 adds
            __builtin_nontemporal_store(s, reinterpret_cast<floatx4*>(r + v));
            a[i][0] = __float_as_uint(s.x);
            a[i][1] = __float_as_uint(s.y);
            a[i][2] = __float_as_uint(s.z);
            a[i][3] = __float_as_uint(s.w);
        }
    } else {
#pragma unroll
        for (int i = 0; i < ITERS; ++i) {
            const uint32_t v = wbase + i * 256 + lane * 4;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                a[i][e] = kAbsent;
                if (v + e >= head && v + e < vend) {
                    const float s = r[v + e] + g[v + e];
                    r[v + e] = s;
                    a[i][e] = present(__float_as_uint(s));
                }
            }
        }
    }

    uint32_t n_in = 0, n_hi = 0, mask = 0, mask_in = 0;          // wave-uniform
    // (the elements of the tail count as candidates and in the histogram, and mark their stretch)
    uint32_t tail_key[3] = {kAbsent, kAbsent, kAbsent}, tail_hi = 0, tail_lo = 0;
    if (has_tail && vgroup > 0u) {                               // wave-uniform
#pragma unroll
        for (int e = 0; e < 3; ++e) {
            if ((uint32_t)e >= head) continue;
            const uint32_t x = (uint32_t)__builtin_amdgcn_readfirstlane((int)a[0][e]);
            if (x != kAbsent) tail_key[e] = present_key(x);
            if (lane == 0) a[0][e] = edge ? kAbsent : kZeroSum;  // (-0.0 is below any other bracket)
            if (tail_key[e] != kAbsent && tail_key[e] >= bk.lo) {
                mask |= 1u;
                if (tail_key[e] >= bk.hi) ++tail_hi; else ++tail_lo;
            }
        }
        if (lane < 3u && vgroup <= gs.ngroups)
            gs.tail[((size_t)w * gs.ngroups + vgroup - 1u) * 3u + lane] = lane == 0 ? tail_key[0] : (lane == 1 ? tail_key[1] : tail_key[2]);
    }
    // reach_lo(x), reach_hi(x): whether the key of x is at or above the bracket's ends
    auto count = [&](auto&& reach_lo, auto&& reach_hi) {
#pragma unroll
        for (int i = 0; i < ITERS; ++i) {
            uint64_t bl[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) bl[e] = __ballot(reach_lo(a[i][e]));
            if ((bl[0] | bl[1] | bl[2] | bl[3]) == 0ull) continue;
            mask |= 1u << i;
            uint32_t in = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const uint32_t h = (uint32_t)__popcll(__ballot(reach_hi(a[i][e])));
                n_hi += h;
                in += (uint32_t)__popcll(bl[e]) - h;
            }
            if (in) mask_in |= 1u << i;
            n_in += in;
        }
    };
    if (!edge)
        count([&](uint32_t x) { return !(__builtin_fabsf(__uint_as_float(x)) < __uint_as_float(bk.lo)); },
              [&](uint32_t x) { return !(__builtin_fabsf(__uint_as_float(x)) < __uint_as_float(bk.hi)); });
    else
        count([&](uint32_t x) { return within(x & kAbs, bk.lo, kAbs); }, [&](uint32_t x) { return within(x & kAbs, bk.hi, kAbs); });
    if (lane == 0) { s_in[wave] = n_in; s_hi[wave] = n_hi; s_mask[wave] = mask; }
    __syncthreads();
    // groups of one repeated key (block-uniform; only where a quarter of the group lies inside the bracket)
    uint32_t grp_in[kGroupsPerBlock], one_key[kGroupsPerBlock];
    bool crowded = false;
#pragma unroll
    for (int q = 0; q < kGroupsPerBlock; ++q) {
        grp_in[q] = 0;
        one_key[q] = kPlainRun;
        for (int v = 0; v < kWavesPerGroup; ++v) grp_in[q] += s_in[q * kWavesPerGroup + v];
        crowded = crowded || grp_in[q] >= kGroup / 4;
    }
    if (crowded) {
        uint32_t mx = 0, mn = kAbs;
#pragma unroll
        for (int i = 0; i < ITERS; ++i)
            if ((mask_in >> i) & 1u)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const uint32_t key = a[i][e] & kAbs;         // (that of kAbsent is above any bracket)
                    if (bk.holds(key)) {
                        mx = key > mx ? key : mx;
                        mn = key < mn ? key : mn;
                    }
                }
        mx = wave_largest(mx);
        mn = kAbs - wave_largest(kAbs - mn);
        if (lane == 0) { s_max[wave] = mx; s_min[wave] = mn; }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < kGroupsPerBlock; ++q) {
            uint32_t x = 0, y = kAbs;
            for (int v = 0; v < kWavesPerGroup; ++v) {
                x = s_max[q * kWavesPerGroup + v] > x ? s_max[q * kWavesPerGroup + v] : x;
                y = s_min[q * kWavesPerGroup + v] < y ? s_min[q * kWavesPerGroup + v] : y;
            }
            if (grp_in[q] != 0u && x == y) one_key[q] = x;
        }
    }
    if (threadIdx.x == 0) {
        uint32_t stored = 0, total = 0;
#pragma unroll
        for (int q = 0; q < kGroupsPerBlock; ++q) stored += one_key[q] == kPlainRun ? grp_in[q] : 0u;
        for (int v = 0; v < kWaves; ++v) total += s_in[v] + s_hi[v];
        uint32_t base = stored ? atomicAdd(&gs.brk_cnt[w], stored) : 0u;
        s_base = base;
        if (total) atomicAdd(&cand_count[w], total);
#pragma unroll
        for (int q = 0; q < kGroupsPerBlock; ++q) {
            const uint32_t grp = chunk * kGroupsPerBlock + q;
            uint32_t above = 0;
            uint64_t mk = 0;
            for (int v = 0; v < kWavesPerGroup; ++v) {
                above += s_hi[q * kWavesPerGroup + v];
                mk |= (uint64_t)s_mask[q * kWavesPerGroup + v] << (v * ITERS);
            }
            if (grp < gs.ngroups)
                gs.run[(size_t)w * gs.ngroups + grp] = make_uint4(base, grp_in[q], above, one_key[q]);
            if (grp <= gs.ngroups) gs.mask[(size_t)w * (gs.ngroups + 1u) + grp] = mk;
            if (one_key[q] == kPlainRun) base += grp_in[q];
        }
    }
    if (lane == 0) {
        if (n_hi + tail_hi) atomicAdd(&s_h[kAboveBin], n_hi + tail_hi);
        if (tail_hi + tail_lo) {
            atomicAdd(&cand_count[w], tail_hi + tail_lo);
#pragma unroll
            for (int e = 0; e < 3; ++e)
                if (tail_key[e] != kAbsent && bk.holds(tail_key[e])) atomicAdd(&s_h[bk.bin(tail_key[e])], 1u);
        }
    }
    __syncthreads();
    const uint32_t my_group = wave / kWavesPerGroup;             // wave-uniform
    uint32_t my_one = kPlainRun;
#pragma unroll
    for (int q = 0; q < kGroupsPerBlock; ++q)
        if ((uint32_t)q == my_group) my_one = one_key[q];
    if (my_one != kPlainRun) {
        if (lane == 0 && n_in) atomicAdd(&s_h[bk.bin(my_one)], n_in);
    } else if (n_in) {
        uint32_t off = s_base;
#pragma unroll
        for (int q = 0; q < kGroupsPerBlock; ++q)
            if ((uint32_t)q < my_group && one_key[q] == kPlainRun) off += grp_in[q];
        for (uint32_t v = my_group * kWavesPerGroup; v < wave; ++v) off += s_in[v];
        float* out = keys + (size_t)w * cap;
        const uint32_t lo = once_more(bk.lo), n = once_more(bk.hi) - lo;
#pragma unroll
        for (int i = 0; i < ITERS; ++i) {
            if (((mask_in >> i) & 1u) == 0u) continue;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const uint32_t rel = (a[i][e] & kAbs) - lo;
                const bool c = rel < n;
                const uint64_t b = __ballot(c);
                if (c) {
                    const uint32_t pos = off + rank_in(b);
                    if (pos < cap) out[pos] = __uint_as_float(rel + lo);
                    atomicAdd(&s_h[rel >> bk.shift], 1u);
                }
                off += (uint32_t)__popcll(b);
            }
        }
    }
    __syncthreads();
    uint32_t* out = gs.hist + (size_t)w * kBrkBins;
    for (int b = threadIdx.x; b < kBrkBins; b += kSBlock) {
        const uint32_t n = s_h[b];
        if (n) atomicAdd(&out[b], n);
    }
}

// ---------------------------------------------------------------------------------
// a group's part of a pair's union
// ---------------------------------------------------------------------------------

// first output position of group g of a set that has been finished (g == ngroups: k)
__device__ __forceinline__ uint32_t group_start(const GroupSets& gs, uint32_t id, uint32_t g) {
    const uint2 o = gs.off[(size_t)id * (gs.ngroups + 1u) + g];
    const uint32_t need = gs.need[id];
    return o.x + (o.y < need ? o.y : need);
}

// Two ways to keep a group's values in registers and LDS:
//   PLAIN   as they are, and -0.0 where there is none: x + -0.0 is x to the bit (for every x that came out of a sum), so
//           the union is one addition, and a key is compared as |value| with a number, one instruction (a NaN is above
//           all, as by its bits).  For groups in which no zero can be selected and no threshold is a NaN: all but a few.
//   !PLAIN  kAbsent where there is none, keys compared as integers; also ranks ties, in the one group of a set in which
//           they run out.
template <bool PLAIN> constexpr uint32_t kNone = PLAIN ? kZeroSum : kAbsent;
template <bool PLAIN>
__device__ __forceinline__ bool reaches(uint32_t v, uint32_t least) {
    if (PLAIN) return !(__builtin_fabsf(__uint_as_float(v)) < __uint_as_float(least));
    return within(v & kAbs, least, kAbs);
}
template <bool PLAIN>
__device__ __forceinline__ uint32_t kept(uint32_t bits) { return PLAIN ? bits : present(bits); }
template <bool PLAIN>
__device__ __forceinline__ uint32_t sum_of(uint32_t a, uint32_t b) {
    if (PLAIN) return __float_as_uint(__uint_as_float(a) + __uint_as_float(b));
    if (a == kAbsent) return b;
    return b == kAbsent ? a : present(__float_as_uint(__uint_as_float(a) + __uint_as_float(b)));
}

// The union of pair p in group g, by index, into LDS: cell c holds the value at index g * kGroup + c, or kNone.
// The value at an index of both operands is their sum (one fp32 add).  s_cell: kGroup words.  Bound by the latency
// of its loads, which two blocks per CU hide from one another.
struct Operands {
    const uint32_t* idx[2];
    const float* val[2];
    uint32_t first[2], end[2];
};
__device__ __forceinline__ Operands group_operands(const GroupSets& gs, const uint32_t* idx, const float* val, uint32_t first_in,
                                                   uint32_t k, uint32_t p, uint32_t g) {
    Operands o;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        o.idx[j] = idx + (size_t)(2u * p + j) * k;
        o.val[j] = val + (size_t)(2u * p + j) * k;
        o.first[j] = group_start(gs, first_in + 2u * p + j, g);
        const uint32_t e = group_start(gs, first_in + 2u * p + j, g + 1u);
        o.end[j] = e < k ? e : k;
    }
    return o;
}
constexpr int kGrpAhead = 4;                  // entries of either operand that a thread loads at once
struct OperandBatch { uint32_t idx[2][kGrpAhead]; float val[2][kGrpAhead]; };
template <int T = kGrpBlock>
__device__ __forceinline__ void load_operand(const Operands& o, int j, uint32_t from, uint32_t (&idx)[kGrpAhead], float (&val)[kGrpAhead]) {
#pragma unroll
    for (int u = 0; u < kGrpAhead; ++u) {
        // (uniform bases, one 32-bit offset)
        const uint32_t first = from + u * T, left = first < o.end[j] ? o.end[j] - first : 0u;
        idx[u] = kAbsent;
        val[u] = 0.0f;
        if (threadIdx.x < left) {
            idx[u] = load_at(o.idx[j] + first, threadIdx.x);
            val[u] = __uint_as_float(load_at(reinterpret_cast<const uint32_t*>(o.val[j]) + first, threadIdx.x));
        }
    }
}
template <bool PLAIN, int T = kGrpBlock>
__device__ __forceinline__ void clear_cells(uint32_t* s_cell) {
#pragma unroll
    for (int u = 0; u < (int)kGroup / T; u += 4)
        *reinterpret_cast<uint4*>(&s_cell[(u / 4 * T + threadIdx.x) * 4]) = make_uint4(kNone<PLAIN>, kNone<PLAIN>, kNone<PLAIN>, kNone<PLAIN>);
}
// b: the operands' first entries, already loaded; the cells hold kNone (seen by every thread only behind the barrier in
// here), and afterwards, behind another one, the union.
template <bool PLAIN, int T = kGrpBlock>
__device__ __forceinline__ void unite(const Operands& o, OperandBatch& b, uint32_t g, uint32_t* s_cell) {
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        if (j) __syncthreads();
        for (uint32_t from = o.first[j];;) {
#pragma unroll
            for (int u = 0; u < kGrpAhead; ++u) {
                const uint32_t c = b.idx[j][u] - g * kGroup;
                if (c >= kGroup) continue;                   // none
                const uint32_t v = kept<PLAIN>(__float_as_uint(b.val[j][u]));
                s_cell[c] = j ? sum_of<PLAIN>(s_cell[c], v) : v;
            }
            from += kGrpAhead * T;
            if (from >= o.end[j]) break;                     // block-uniform
            load_operand<T>(o, j, from, b.idx[j], b.val[j]);
        }
    }
    __syncthreads();
}

// ---------------------------------------------------------------------------------
// the walk of the bracket's keys, and the next round's bracket
// ---------------------------------------------------------------------------------

// The sets of one launch.
struct GroupBatch {
    uint32_t first;             // number of the first set
    uint32_t k;
    const uint32_t* keys;       // bracket keys, rows key_stride apart
    size_t key_stride;
    uint2* list;                // [sets][list_cap] in-bin entries: key, group | count << 12
    uint32_t list_cap;
    uint32_t keys_cap;          // workers: keys a row holds (more were counted than stored: missed); pairs: never
    const float* rows;          // workers: the accumulated rows (NULL: the sets are pairs)
    int64_t stride;
    const uint32_t* in_idx;     // pairs: operands 2 p and 2 p + 1, k entries each
    const float* in_val;
    uint32_t first_in;          // pairs: number of operand 0
};
// sample of the unions of the NEXT round's pairs and the bracket it gives
struct GroupSample {
    uint32_t next_first;        // number of the first of these pairs
    uint32_t pairs;             // 0: no next round
    const uint32_t* samples;    // [sets][n] sampled values of this launch's sets, at the same indices (kAbsent: none)
    uint32_t n;
    uint32_t target_lo, target_hi;
};

constexpr int kGrpWalkBlock = 1024;
constexpr int kGrpWalkRuns = 2;           // groups per wave
constexpr uint32_t kGrpWeightShift = 13;
static_assert(kMaxIndexGroups <= 1u << kGrpWeightShift && kGroup + 3 < 1u << (32 - kGrpWeightShift), "a list entry's fields");

// Bin of the k-th key of set `id` (kMissed: outside the bracket) and its rank in there; every thread calls it.
__device__ __forceinline__ uint32_t pick_bin(const GroupSets& gs, uint32_t id, uint32_t k, uint32_t* s_wave, uint32_t* s_out,
                                             uint32_t& krem) {
    constexpr int kPer = kBrkBins / kGrpWalkBlock;
    uint32_t loc[kPer];
#pragma unroll
    for (int j = 0; j < kPer; ++j) loc[j] = gs.hist[(size_t)id * kBrkBins + threadIdx.x * kPer + j];
    suffix_pick<kPer>(loc, k, s_wave, s_out);
    krem = k - s_out[1];
    return s_out[2] == 0u || s_out[0] == kAboveBin ? kMissed : s_out[0];
}

// Bracket of pair blockIdx.y of the next round, from a sample of its union: each operand as it will be, cut off
// at the lower edge of its k-th key's bin (the exact key is a fraction of a permille off).
__device__ inline void pick_bracket(const GroupSets& gs, const GroupBatch& gb, const GroupSample& sm, uint32_t* h,
                                    uint32_t* s_wave, uint32_t* s_out) {
    const uint32_t p = blockIdx.y, t = threadIdx.x;
    for (int b = t; b < kSampleBins; b += kGrpWalkBlock) h[b] = 0u;
    uint32_t T[2];
#pragma unroll
    for (int side = 0; side < 2; ++side) {
        const uint32_t id = gb.first + 2u * p + side;
        uint32_t krem;
        const uint32_t d = pick_bin(gs, id, gb.k, s_wave, s_out, krem);
        T[side] = d == kMissed ? (s_out[2] == 0u ? 0u : gs.hi[id]) : Bracket(gs, id).bin_lo(d);
        __syncthreads();
    }
    const uint32_t n = sm.n;
    const uint32_t* sx = sm.samples + (size_t)(2u * p) * n;
    const uint32_t* sy = sx + n;
    constexpr int kU = 16;
    for (uint32_t i0 = 0; i0 < n; i0 += kGrpWalkBlock * kU) {
        uint32_t x[kU], y[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const uint32_t i = i0 + u * kGrpWalkBlock + t;
            x[u] = i < n ? sx[i] : kAbsent;
            y[u] = i < n ? sy[i] : kAbsent;
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const bool hx = x[u] != kAbsent && (x[u] & kAbs) >= T[0], hy = y[u] != kAbsent && (y[u] & kAbs) >= T[1];
            if (!hx && !hy) continue;
            const float v = hx && hy ? __uint_as_float(x[u]) + __uint_as_float(y[u]) : __uint_as_float(hx ? x[u] : y[u]);
            atomicAdd(&h[(__float_as_uint(v) & kAbs) >> kSampleShift], 1u);
        }
    }
    __syncthreads();
    constexpr int kPer = kSampleBins / kGrpWalkBlock;
    uint32_t loc[kPer];
#pragma unroll
    for (int j = 0; j < kPer; ++j) loc[j] = h[t * kPer + j];
    suffix_pick<kPer>(loc, sm.target_lo, s_wave, s_out);
    const uint32_t lo = s_out[2] ? s_out[0] << kSampleShift : 0u;
    __syncthreads();
    suffix_pick<kPer>(loc, sm.target_hi + 1u, s_wave, s_out);
    if (t == 0) {
        const uint32_t hi = s_out[2] ? (s_out[0] + 1u) << kSampleShift : 1u << kSampleShift;
        gs.lo[sm.next_first + p] = lo < kInfKey ? lo : kInfKey;
        gs.hi[sm.next_first + p] = hi < kInfKey ? hi : kInfKey;
    }
}

// A set that missed its bracket: the blocks of its row share its groups, count the top digit of every key (the bracket
// that k_group_finish takes instead) and, of a pair, store the keys where those of the bracket would be.
// h: kTopBins + kGroup words of LDS.
__device__ inline void count_all(const GroupSets& gs, const GroupBatch& gb, uint32_t id, uint32_t* h) {
    const uint32_t t = threadIdx.x, p = blockIdx.y;
    uint32_t* s_cell = h + kTopBins;
    for (uint32_t b = t; b < kTopBins; b += kGrpWalkBlock) h[b] = 0u;
    __syncthreads();
    auto count = [&](uint32_t key) {                         // (masses of one key: added once)
        const uint64_t act = __ballot(key != kAbsent);
        if (!act) return;
        const uint32_t b = key >> 20, first = (uint32_t)__builtin_ctzll(act);
        if (__ballot(key != kAbsent && b == lane_value(b, first)) == act) {
            if (lane_id() == first) atomicAdd(&h[b], (uint32_t)__popcll(act));
        } else if (key != kAbsent) {
            atomicAdd(&h[b], 1u);
        }
    };
    if (gb.rows) {                                           // a wave per stretch of 1024 elements
        constexpr int kU = 16;
        const float* row = gb.rows + (int64_t)p * gb.stride;
        constexpr uint32_t kStretch = kWave * kU;
        for (uint32_t i0 = ((blockIdx.x - 1u) * (kGrpWalkBlock / kWave) + t / kWave) * kStretch; i0 < gs.m;
             i0 += (gridDim.x - 1u) * (kGrpWalkBlock / kWave) * kStretch) {
            uint32_t key[kU];
#pragma unroll
            for (int j = 0; j < kU; ++j) {
                const uint32_t i = i0 + j * kWave + lane_id();
                const uint32_t x = __float_as_uint(row[i < gs.m ? i : 0u]);      // (in flight together, see finish_set)
                key[j] = i < gs.m ? present_key(x) : kAbsent;
            }
#pragma unroll
            for (int j = 0; j < kU; ++j) count(key[j]);
        }
    }
    for (uint32_t g = blockIdx.x - 1u; !gb.rows && g < gs.ngroups; g += gridDim.x - 1u) {
        const Operands o = group_operands(gs, gb.in_idx, gb.in_val, gb.first_in, gb.k, p, g);
        OperandBatch b;
        load_operand<kGrpWalkBlock>(o, 0, o.first[0], b.idx[0], b.val[0]);
        load_operand<kGrpWalkBlock>(o, 1, o.first[1], b.idx[1], b.val[1]);
        clear_cells<false, kGrpWalkBlock>(s_cell);
        unite<false, kGrpWalkBlock>(o, b, g, s_cell);
        constexpr int kPer = (int)kGroup / kGrpWalkBlock;
        uint32_t key[kPer];
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            const uint32_t v = s_cell[j * kGrpWalkBlock + t];
            key[j] = v == kAbsent ? kAbsent : v & kAbs;
        }
#pragma unroll
        for (int j = 0; j < kPer; ++j) count(key[j]);
        __syncthreads();                                     // the cells have been read
        if (t == 0) s_cell[0] = 0u;
        __syncthreads();
        const uint32_t region = o.first[0] + o.first[1];
        uint32_t* keys = const_cast<uint32_t*>(gb.keys) + (size_t)p * gb.key_stride;
#pragma unroll
        for (int j = 0; j < kPer; ++j)
            if (key[j] != kAbsent) {
                const uint32_t at = region + atomicAdd(&s_cell[0], 1u);
                if (at < gb.key_stride) keys[at] = key[j];
            }
        __syncthreads();
        if (t == 0) gs.run[(size_t)id * gs.ngroups + g] = make_uint4(region, s_cell[0], 0u, kPlainRun);
        __syncthreads();
    }
    __syncthreads();
    for (uint32_t b = t; b < kTopBins; b += kGrpWalkBlock)
        if (h[b]) atomicAdd(&gs.hist_all[(size_t)id * kAllBins + b], h[b]);
}

// Block 0 of row p: the next round's pair p; blocks from 1 on: sixteen waves with kGrpWalkRuns groups each of set p.
// The list is short (tens of keys to a few thousand): the keys of a run that are all one key are one entry.
// Two groups per wave: 69 us for the 32 workers' sets at m = 25,557,032, k = 6.4 M; one 97, four 88 (the longest runs bound it).
// Long runs (hot layers that hold most of the bracket's keys) are read sixteen loads at a time: m = 1.05 M, P = 16, k = m / 4, ten
// layers 33 .. 26 -> 23 .. 18 us a launch (four loads, and one in the second walk, before).
__global__ __launch_bounds__(kGrpWalkBlock) void k_group_walk(GroupSets gs, GroupBatch gb, GroupSample sm) {
    constexpr int kWaves = kGrpWalkBlock / kWave;
    constexpr uint32_t kStash = 64;                          // entries a wave parks
    __shared__ uint32_t h[kSampleBins];
    __shared__ uint32_t s_wave[kWaves];
    __shared__ uint32_t s_out[3];
    __shared__ uint32_t s_cnt[kWaves];
    __shared__ uint32_t s_base;
    if (blockIdx.x == 0) {
        if (blockIdx.y < sm.pairs) pick_bracket(gs, gb, sm, h, s_wave, s_out);
        return;
    }
    const uint32_t id = gb.first + blockIdx.y;
    const uint32_t lane = lane_id(), wave = threadIdx.x / kWave;
    const uint32_t g0 = ((blockIdx.x - 1u) * kWaves + wave) * kGrpWalkRuns;
    const uint32_t* keys = gb.keys + (size_t)blockIdx.y * gb.key_stride;
    // (the runs' first keys are fetched in front of the pick, which hides their latency)
    constexpr int kU = 4, kBatch = 16;
    uint4 runs[kGrpWalkRuns];
    uint32_t ahead[kGrpWalkRuns][kU];
#pragma unroll
    for (int q = 0; q < kGrpWalkRuns; ++q)
        runs[q] = g0 + q < gs.ngroups ? gs.run[(size_t)id * gs.ngroups + g0 + q] : make_uint4(0u, 0u, 0u, kPlainRun);
#pragma unroll
    for (int q = 0; q < kGrpWalkRuns; ++q)
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const uint32_t i = u * kWave + lane;
            ahead[q][u] = i < runs[q].y && runs[q].w == kPlainRun && runs[q].x + i < gb.key_stride ? keys[runs[q].x + i] : kAbsent;
        }
    uint32_t krem;
    const uint32_t d1 = pick_bin(gs, id, gb.k, s_wave, s_out, krem);
    // (a list holds as many entries as a row's stored keys: four of a group may come on top of those, its tail and its one key)
    const bool missed = d1 == kMissed || (gb.rows && gs.brk_cnt[id] + 4u * gs.ngroups > gb.keys_cap);      // block-uniform
    if (blockIdx.x == 1 && threadIdx.x == 0) {
        gs.d1[id] = missed ? kMissed : d1;
        gs.krem[id] = krem;
    }
    if (missed) {
        count_all(gs, gb, id, h);
        return;
    }
    const Bracket bk(gs, id);
    const uint32_t head = gb.rows ? (uint32_t)(((int64_t)blockIdx.y * gb.stride) & 3) : 0u;
    uint2* list = gb.list + (size_t)blockIdx.y * gb.list_cap;
    uint2* stash = reinterpret_cast<uint2*>(h) + wave * kStash;
    uint32_t nst = 0;                                        // wave-uniform: entries parked
#pragma unroll
    for (int q = 0; q < kGrpWalkRuns; ++q) {
        const uint32_t g = g0 + q;
        if (g >= gs.ngroups) break;                          // wave-uniform
        const uint4 run = runs[q];
        uint32_t gt = run.z, mx = 0, mn = kAbs, in = 0, own_gt = 0;
        const bool plain = run.w == kPlainRun;
        // keys [i0, i0 + 64 kBatch) of the run, a lane's in step
        uint32_t key[kBatch];
        auto load = [&](uint32_t i0) {
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                const uint32_t i = i0 + u * kWave + lane, x = keys[run.x + (i < run.y ? i : 0u)];
                key[u] = i < run.y ? x : kAbsent;
            }
        };
        // (the row's last elements on v belong to this group: up to three keys of their own)
        uint32_t tk = kAbsent;
        if (head && lane < 3u && ((uint64_t)(g + 1u) << kGroupLog2) < (uint64_t)gs.m + head)
            tk = gs.tail[((size_t)blockIdx.y * gs.ngroups + g) * 3u + lane];
        if (tk != kAbsent) {
            if (tk >= bk.hi) ++own_gt;
            else if (tk >= bk.lo) {
                const uint32_t b = bk.bin(tk);
                if (b > d1) ++own_gt;
                else if (b == d1) { ++in; mx = tk; mn = tk; }
            }
        }
        if (plain) {
            auto see = [&](uint32_t x) {
                if (x == kAbsent) return;
                const uint32_t b = bk.bin(x);
                if (b > d1) ++own_gt;
                else if (b == d1) {
                    ++in;
                    mx = x > mx ? x : mx;
                    mn = x < mn ? x : mn;
                }
            };
#pragma unroll
            for (int u = 0; u < kU; ++u) see(ahead[q][u]);
            for (uint32_t i0 = kWave * kU; i0 < run.y; i0 += kWave * kBatch) {
                load(i0);
#pragma unroll
                for (int u = 0; u < kBatch; ++u) see(key[u]);
            }
        } else if (lane == 0) {
            const uint32_t b = bk.bin(run.w);
            if (b > d1) own_gt += run.y;
            else if (b == d1) {
                in += run.y;
                mx = run.w > mx ? run.w : mx;
                mn = run.w < mn ? run.w : mn;
            }
        }
        own_gt = wave_total(own_gt);
        in = wave_total(in);
        mx = wave_largest(mx);
        mn = kAbs - wave_largest(kAbs - mn);
        gt += own_gt;
        if (lane == 0) gs.grp_gt[(size_t)id * gs.ngroups + g] = gt;
        if (in == 0u) continue;
        // entries of this run: one if its keys agree (always so for a run of one key without a tail), else each key of its
        // own (a run of one key beside a tail of others: one for the run)
        const bool one = mx == mn, tail_in = tk != kAbsent && bk.holds(tk) && bk.bin(tk) == d1, run_in = !plain && bk.bin(run.w) == d1;
        const uint32_t entries = one ? 1u : (plain ? in : (uint32_t)__popcll(__ballot(tail_in)) + (run_in ? 1u : 0u));
        uint32_t pos = nst;                                  // in the stash, or straight in the list
        const bool parked = nst + entries <= kStash;
        uint2* dst = stash;
        uint32_t room = kStash;
        if (parked) nst += entries;
        else {
            uint32_t b = 0;
            if (lane == 0) b = atomicAdd(&gs.list_cnt[id], entries);
            pos = lane_value(b, 0u);
            dst = list;
            room = gb.list_cap;
        }
        if (one) {
            if (lane == 0 && pos < room) dst[pos] = make_uint2(mx, g | in << kGrpWeightShift);
            continue;
        }
        auto put = [&](bool c, uint32_t key, uint32_t weight) {
            const uint64_t b = __ballot(c);
            if (c) {
                const uint32_t at = pos + rank_in(b);
                if (at < room) dst[at] = make_uint2(key, g | weight << kGrpWeightShift);
            }
            pos += (uint32_t)__popcll(b);
        };
        put(tail_in, tk, 1u);
        if (plain) {
            for (uint32_t i0 = 0; i0 < run.y; i0 += kWave * kBatch) {
                load(i0);
#pragma unroll
                for (int u = 0; u < kBatch; ++u) put(key[u] != kAbsent && bk.bin(key[u]) == d1, key[u], 1u);
            }
        } else {
            put(lane == 0 && run_in, run.w, run.y);
        }
    }
    if (lane == 0) s_cnt[wave] = nst;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t n = 0;
        for (int v = 0; v < kWaves; ++v) n += s_cnt[v];
        s_base = n ? atomicAdd(&gs.list_cnt[id], n) : 0u;    // one reservation per block
    }
    __syncthreads();
    uint32_t pos = s_base;
    for (uint32_t v = 0; v < wave; ++v) pos += s_cnt[v];
    if (lane < nst && pos + lane < gb.list_cap) list[pos + lane] = stash[lane];
}

// ---------------------------------------------------------------------------------
// exact key, ties to take, output positions of the groups
// ---------------------------------------------------------------------------------

constexpr int kGrpFinishBlock = 1024;

// All keys of group g of a set that missed its bracket: where they lie and how many there are.
__device__ __forceinline__ uint32_t group_keys(const GroupSets& gs, const GroupBatch& gb, uint32_t p, uint32_t g, const uint32_t*& from) {
    if (gb.rows) {
        from = reinterpret_cast<const uint32_t*>(gb.rows) + (int64_t)p * gb.stride + (size_t)g * kGroup;
        return gs.m - g * kGroup < kGroup ? gs.m - g * kGroup : kGroup;
    }
    const uint4 run = gs.run[(size_t)(gb.first + p) * gs.ngroups + g];
    from = gb.keys + (size_t)p * gb.key_stride + run.x;
    return run.y;
}

// A set that missed its bracket gets another one, which holds the k-th key for certain: the top digit `top` that all its
// keys' histogram gives.  Its blocks share its groups, a wave per group: keys above are counted, those inside listed as
// k_group_walk would (1024 elements whose keys agree are one entry) and their next ten bits histogrammed.
// A wave goes over its group twice, so that the block reserves room for sixteen groups at once.  h: 1024 words of LDS,
// s_cnt: two rows of a word per wave and one more.
__device__ inline void collect_missed(const GroupSets& gs, const GroupBatch& gb, uint32_t p, uint32_t top, uint32_t* h, uint32_t* s_cnt) {
    constexpr int kU = 16;
    constexpr uint32_t kWaves = kGrpFinishBlock / kWave, kTurns = kGroup / (kWave * kU);
    const uint32_t id = gb.first + p, t = threadIdx.x, lane = lane_id(), wave = t / kWave;
    uint2* list = gb.list + (size_t)p * gb.list_cap;
    h[t] = 0u;
    uint32_t* cnt = s_cnt;
    for (uint32_t g0 = blockIdx.y * kWaves; g0 < gs.ngroups; g0 += gridDim.y * kWaves) {         // block-uniform
        const uint32_t g = g0 + wave;
        const uint32_t* from = nullptr;
        const uint32_t count = g < gs.ngroups ? group_keys(gs, gb, p, g, from) : 0u;
        uint32_t key[kU];
        auto load = [&](uint32_t turn) {
#pragma unroll
            for (int j = 0; j < kU; ++j) {
                const uint32_t i = turn * (kWave * kU) + j * kWave + lane;
                const uint32_t x = from[i < count ? i : 0u];
                key[j] = i < count ? present_key(x) : kAbsent;
            }
        };
        // (all wave-uniform) keys above, entries; turns with any, turns whose keys agree
        uint32_t gt = 0, entries = 0, some = 0, agree = 0;
        for (uint32_t turn = 0; turn < kTurns && turn * (kWave * kU) < count; ++turn) {
            load(turn);
            uint32_t in = 0, mx = 0, mn = kAbs;
#pragma unroll
            for (int j = 0; j < kU; ++j) {
                const uint32_t d = key[j] >> 20;
                gt += (uint32_t)__popcll(__ballot(key[j] != kAbsent && d > top));
                in += (uint32_t)__popcll(__ballot(d == top));
                if (d == top) {
                    mx = key[j] > mx ? key[j] : mx;
                    mn = key[j] < mn ? key[j] : mn;
                }
            }
            if (in == 0u) continue;
            some |= 1u << turn;
            const bool one = wave_largest(mx) == kAbs - wave_largest(kAbs - mn);
            agree |= one ? 1u << turn : 0u;
            entries += one ? 1u : in;
        }
        if (lane == 0) {
            cnt[wave] = entries;
            if (g < gs.ngroups) gs.grp_gt[(size_t)id * gs.ngroups + g] = gt;
        }
        __syncthreads();
        const uint32_t all = row_incl_scan(lane < kWaves ? cnt[lane] : 0u);
        if (t == 0) s_cnt[2 * kWaves] = atomicAdd(&gs.list_cnt[id], lane_value(all, kWaves - 1u));
        __syncthreads();
        uint32_t pos = s_cnt[2 * kWaves] + lane_value(all, wave) - entries;
        for (uint32_t turn = 0; turn < kTurns; ++turn) {
            if (((some >> turn) & 1u) == 0u) continue;
            load(turn);
            if ((agree >> turn) & 1u) {
                uint32_t in = 0, mx = 0;
#pragma unroll
                for (int j = 0; j < kU; ++j) {
                    const bool c = key[j] >> 20 == top;
                    in += (uint32_t)__popcll(__ballot(c));
                    mx = c ? key[j] : mx;
                }
                mx = wave_largest(mx);
                if (lane == 0) {
                    if (pos < gb.list_cap) list[pos] = make_uint2(mx, g | in << kGrpWeightShift);
                    atomicAdd(&h[(mx >> 10) & 1023u], in);
                }
                ++pos;
                continue;
            }
#pragma unroll
            for (int j = 0; j < kU; ++j) {
                const bool c = key[j] >> 20 == top;
                const uint64_t b = __ballot(c);
                if (c) {
                    const uint32_t at = pos + rank_in(b);
                    if (at < gb.list_cap) list[at] = make_uint2(key[j], g | 1u << kGrpWeightShift);
                    atomicAdd(&h[(key[j] >> 10) & 1023u], 1u);
                }
                pos += (uint32_t)__popcll(b);
            }
        }
        cnt = cnt == s_cnt ? s_cnt + kWaves : s_cnt;         // (the other row may still be read)
    }
    __syncthreads();
    const uint32_t n = h[t];
    if (n) atomicAdd(&gs.hist_all[(size_t)id * kAllBins + kTopBins + t], n);
}

struct FinishShared {
    uint32_t h[2048];
    uint32_t g_gt[kMaxIndexGroups], g_eq[kMaxIndexGroups];
    uint32_t wave[kGrpFinishBlock / kWave];
    uint32_t out[3];
    uint32_t turn, cnt[2 * (kGrpFinishBlock / kWave) + 1];
};
// The exact key, the ties and the groups' output positions of set p from its list of n entries: the keys in
// [base, base + width), among which the k-th has rank krem.  MISSED: a long list, see collect_missed.
template <bool MISSED>
__device__ __forceinline__ void finish_set(FinishShared& sh, const GroupSets& gs, const GroupBatch& gb, uint32_t p, uint32_t base,
                                           uint32_t width, uint32_t krem, uint32_t n) {
    constexpr int kT = kGrpFinishBlock;
    constexpr int kPer = (int)(kMaxIndexGroups / kT);
    uint32_t* h = sh.h;
    uint32_t* g_gt = sh.g_gt;
    uint32_t* g_eq = sh.g_eq;
    uint32_t* s_wave = sh.wave;
    uint32_t* s_out = sh.out;
    const uint32_t id = gb.first + p, t = threadIdx.x;
    const uint2* list = gb.list + (size_t)p * gb.list_cap;
    const uint32_t* all = gs.hist_all + (size_t)id * kAllBins;
    // (masses of few keys: the list of a row may not hold them, then all of its keys are read)
    const bool whole = MISSED && n > gb.list_cap;            // block-uniform
    // (every load from an address that is there, so that none waits for the one before: eight in turn took 3 us)
    const uint32_t* grp_gt = gs.grp_gt + (size_t)id * gs.ngroups;
    uint32_t above[kPer];
#pragma unroll
    for (int j = 0; j < kPer; ++j) above[j] = grp_gt[t + j * kT < gs.ngroups ? t + j * kT : 0u];
    // f(key, group, count) for every entry that may be the k-th: the list, or of a set that it does not hold all
    // there are.  The lanes of a wave call f in step; key == kAbsent: nothing.
    constexpr int kCache = 4, kAhead = MISSED ? 16 : kCache;
    uint2 e[kCache];
    const bool cached = n <= (uint32_t)(kCache * kT);
#pragma unroll
    for (int j = 0; j < kCache; ++j) {
        const uint32_t i = j * kT + t;
        e[j] = list[i < n ? i : 0u];
        if (!cached || i >= n) e[j] = make_uint2(kAbsent, 0u);
    }
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const uint32_t g = t + j * kT;
        g_gt[g] = g < gs.ngroups && !whole ? above[j] : 0u;
        g_eq[g] = 0u;
    }
    auto entry = [&](const uint2& x, auto&& f) { f(x.x, x.y & (kMaxIndexGroups - 1u), x.y >> kGrpWeightShift); };
    auto each = [&](auto&& f) {
        if (cached) {
#pragma unroll
            for (int j = 0; j < kCache; ++j) entry(e[j], f);
        } else if (!whole) {
            for (uint32_t i0 = 0; i0 < n; i0 += kT * kAhead) {
                uint2 x[kAhead];
#pragma unroll
                for (int j = 0; j < kAhead; ++j) {
                    const uint32_t i = i0 + j * kT + t;
                    x[j] = list[i < n ? i : 0u];
                    if (i >= n) x[j] = make_uint2(kAbsent, 0u);
                }
#pragma unroll
                for (int j = 0; j < kAhead; ++j) entry(x[j], f);
            }
        } else {
            // a wave per group; f is called in step within a wave
            constexpr int kU = 16;
            for (uint32_t g = t / kWave; g < gs.ngroups; g += kT / kWave) {
                const uint32_t* from;
                const uint32_t count = group_keys(gs, gb, p, g, from);
                for (uint32_t i0 = 0; i0 < count; i0 += kWave * kU) {
                    uint32_t x[kU];
#pragma unroll
                    for (int j = 0; j < kU; ++j) {
                        const uint32_t i = i0 + j * kWave + lane_id();
                        const uint32_t y = from[i < count ? i : 0u];
                        x[j] = i < count ? present_key(y) : kAbsent;
                    }
#pragma unroll
                    for (int j = 0; j < kU; ++j) f(x[j], g, 1u);
                }
            }
        }
    };
    // radix passes over key - base: bits 30..20, 19..10, 9..0; a pass whose bits are zero throughout is skipped
    if (whole) {
        base = 0u;
        width = 0x80000000u;
        krem = gb.k;
    }
    // (of a set that missed its bracket the list is long, a group's entries behind one another: added once per wave)
    auto count_above = [&](bool c, uint32_t g, uint32_t count) {
        const uint64_t act = __ballot(c);
        if (!act) return;
        const uint32_t first = (uint32_t)__builtin_ctzll(act), g0 = lane_value(g, first);
        if (__ballot(c && g == g0 && count == 1u) == act) {
            if (lane_id() == first) atomicAdd(&g_gt[g0], (uint32_t)__popcll(act));
        } else if (c) {
            atomicAdd(&g_gt[g], count);
        }
    };
    uint32_t prefix = 0;
    for (int pass = 0; pass < 3; ++pass) {
        const int shift = pass == 0 ? 20 : (pass == 1 ? 10 : 0);
        const int bits = pass == 0 ? 11 : 10;
        if (shift > 0 && width <= (1u << shift)) continue;   // uniform
        // (of a set that missed its bracket the walk has counted these, or the collecting blocks have)
        const bool counted = whole ? pass == 0 : MISSED && pass == 1;
        h[t] = counted ? all[pass * kTopBins + t] : 0u;
        h[t + kT] = counted && pass == 0 ? all[t + kT] : 0u;
        __syncthreads();
        if (!counted) each([&](uint32_t key, uint32_t g, uint32_t count) {
            const uint32_t rel = key - base, digits = rel >> (shift + bits);
            const bool mine = key != kAbsent && key >= base && digits == prefix;
            if (MISSED && !whole) count_above(key != kAbsent && digits > prefix, g, count);
            const uint32_t b = (rel >> shift) & ((1u << bits) - 1u);
            const uint64_t act = __ballot(mine);
            if (!act) return;
            // (masses of one key: added once)
            const uint32_t first = (uint32_t)__builtin_ctzll(act), b0 = lane_value(b, first);
            if (whole && __ballot(mine && b == b0) == act) {
                if (lane_id() == first) atomicAdd(&h[b0], (uint32_t)__popcll(act));
            } else if (mine) {
                atomicAdd(&h[b], count);
            }
        });
        __syncthreads();
        const uint32_t loc[2] = {h[2 * t], h[2 * t + 1]};
        suffix_pick<2>(loc, krem, s_wave, s_out);
        prefix = (prefix << bits) | s_out[0];
        krem -= s_out[1];
        __syncthreads();
    }
    const uint32_t T = base + prefix, need = krem;
    each([&](uint32_t key, uint32_t g, uint32_t count) {
        if (whole) {                                         // one group per wave
            const uint64_t a = __ballot(key != kAbsent && key > T), q = __ballot(key == T);
            if (lane_id() == 0 && a) atomicAdd(&g_gt[g], (uint32_t)__popcll(a));
            if (lane_id() == 0 && q) atomicAdd(&g_eq[g], (uint32_t)__popcll(q));
        } else if (MISSED) {                                 // (those above the k-th key's second digit have been counted)
            if (key == kAbsent || (key - base) >> 10 != prefix >> 10) return;
            if (key > T) atomicAdd(&g_gt[g], count);
            else if (key == T) atomicAdd(&g_eq[g], count);
        } else if (key != kAbsent) {
            if (key > T) atomicAdd(&g_gt[g], count);
            else if (key == T) atomicAdd(&g_eq[g], count);
        }
    });
    __syncthreads();
    uint32_t a[kPer], q[kPer], sa = 0, sq = 0;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        a[j] = g_gt[t * kPer + j];
        q[j] = g_eq[t * kPer + j];
        sa += a[j];
        sq += q[j];
    }
    uint32_t tot;
    uint32_t ia = block_incl_scan(sa, s_wave, tot) - sa, iq = block_incl_scan(sq, s_wave, tot) - sq;
    uint2* off = gs.off + (size_t)id * (gs.ngroups + 1u);
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const uint32_t g = t * kPer + j;
        if (g <= gs.ngroups) off[g] = make_uint2(ia, iq);
        ia += a[j];
        iq += q[j];
    }
    // (every entry holds running totals, the last one too: group_cut takes differences for the groups' ties)
    if (t == kT - 1 && gs.ngroups == kMaxIndexGroups) off[gs.ngroups] = make_uint2(ia, iq);
    if (t == 0) {
        gs.T[id] = T;
        gs.need[id] = need;
    }
}

// Block (p, 0): set p of the batch, bound by its chain of loads and barriers (6 to 11 us).  The set's other blocks return at
// once unless it missed its bracket: then they share its groups, and the last of them to be done with its part goes on as
// block 0 does.  No block waits for another.
__global__ __launch_bounds__(kGrpFinishBlock) void k_group_finish(GroupSets gs, GroupBatch gb) {
    __shared__ FinishShared sh;
    const uint32_t p = blockIdx.x, id = gb.first + p, t = threadIdx.x;
    const uint32_t d1 = gs.d1[id];
    uint32_t krem = gs.krem[id], n = gs.list_cnt[id];
    const Bracket bk(gs, id);
    if (d1 != kMissed) {                                     // block-uniform
        if (blockIdx.y == 0) finish_set<false>(sh, gs, gb, p, bk.bin_lo(d1), 1u << bk.shift, krem, n);
        return;
    }
    const uint32_t* all = gs.hist_all + (size_t)id * kAllBins;
    const uint32_t loc[2] = {all[2 * t], all[2 * t + 1]};
    suffix_pick<2>(loc, gb.k, sh.wave, sh.out);
    const uint32_t top = sh.out[0];
    krem = gb.k - sh.out[1];
    collect_missed(gs, gb, p, top, sh.h, sh.cnt);
    // (every wave's stores have reached the L2 before the block meets; then one fence writes them back for the last block,
    // which may sit on another XCD)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (t == 0) {
        __threadfence();
        sh.turn = atomicAdd(&gs.arrived[id], 1u);
    }
    __syncthreads();
    if (sh.turn != gridDim.y - 1u) return;                   // block-uniform
    __threadfence();
    n = __hip_atomic_load(&gs.list_cnt[id], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    finish_set<true>(sh, gs, gb, p, top << 20, 1u << 20, krem, n);
}

// ---------------------------------------------------------------------------------
// select and merge
// ---------------------------------------------------------------------------------

// Where a group's part of a set is cut off and where it goes: entries with key >= least are selected; `ranked` (the one
// group of a set in which the ties run out): of those equal to `least` only the first `ties`.
struct GroupCut {
    uint32_t least, out, ties;  // out: first output position
    bool ranked;
};
__device__ __forceinline__ GroupCut group_cut(const GroupSets& gs, uint32_t id, uint32_t g) {
    const uint2* off = gs.off + (size_t)id * (gs.ngroups + 1u) + g;
    const uint2 o = off[0];
    const uint32_t T = gs.T[id], need = gs.need[id], here = off[1].y - o.y, before = o.y < need ? o.y : need;
    const uint32_t ties = need - before;
    return GroupCut{ties >= here ? T : (ties ? T : T + 1u), o.x + before, ties, ties != 0u && ties < here};
}
// Whether the group may be kept PLAIN.
__device__ __forceinline__ bool plain_cut(const GroupCut& c) { return !c.ranked && c.least - 1u < kInfKey; }

// `live`, here and below: which quarters of this wave's sixteen steps hold anything; uniform.  f is called with each
// live step's number, as a constant.
template <int J> struct Step { static constexpr int j = J; };
template <int Q = 0, class F>
__device__ __forceinline__ void for_live_steps(uint32_t live, F&& f) {
    if ((live >> Q) & 1u) {
        f(Step<4 * Q>{});
        f(Step<4 * Q + 1>{});
        f(Step<4 * Q + 2>{});
        f(Step<4 * Q + 3>{});
    }
    if constexpr (Q < 3) for_live_steps<Q + 1>(live, f);
}
static_assert(kGrpPer == 16, "four quarters");
// Lane J of (lo, hi) becomes the uniform mask m.  (The wait states between a comparison that writes m and an
// instruction that reads it are in the block: the compiler does not look into it.)
template <int J>
__device__ __forceinline__ void set_lane(uint32_t& lo, uint32_t& hi, uint64_t m) {
    asm("s_nop 3\n\tv_writelane_b32 %0, %2, %4\n\tv_writelane_b32 %1, %3, %4"
        : "+v"(lo), "+v"(hi) : "s"((uint32_t)m), "s"((uint32_t)(m >> 32)), "n"(J));
}
// n + the number of set bits of `mask` below the calling lane
__device__ __forceinline__ uint32_t rank_from(uint64_t mask, uint32_t n) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, n));
}

// Sum over the lanes below kGrpWaves (x: 0 in all others); uniform.
__device__ __forceinline__ uint32_t few_lanes_sum(uint32_t x) {
    static_assert(kGrpWaves <= 16, "a row of lanes");
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0xB1, 0xf, 0xf, true);       // quad_perm [1,0,3,2]
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x4E, 0xf, 0xf, true);       // quad_perm [2,3,0,1]
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x141, 0xf, 0xf, true);      // row_half_mirror
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x140, 0xf, 0xf, true);      // row_mirror
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)x);
}

// Entries of this wave's 1024 elements at or above the cut / (ranked) equal to it.
template <bool PLAIN>
__device__ __forceinline__ uint2 count_cut(const uint32_t (&v)[kGrpPer], uint32_t live, const GroupCut& c) {
    uint32_t n = 0, eq = 0;
    for_live_steps(once_more(live), [&](auto step) {
        constexpr int j = decltype(step)::j;
        n += (uint32_t)__popcll(__ballot(reaches<PLAIN>(v[j], c.least)));
        if (!PLAIN && c.ranked) eq += (uint32_t)__popcll(__ballot((v[j] & kAbs) == c.least));
    });
    return make_uint2(n, eq);
}
// Writes this wave's selected elements in index order (lane = element: whole rows of stores) and makes the others
// kNone.  counts: count_cut of every wave.  Returns, in lane j < 16, the mask of the elements selected in step j.
template <bool PLAIN, bool DIVIDE>
__device__ __forceinline__ uint64_t emit_cut(uint32_t (&v)[kGrpPer], uint32_t live, const GroupCut& c, const uint2* counts,
                                             uint32_t first_index, uint32_t k, uint32_t* __restrict__ out_idx,
                                             float* __restrict__ out_val, float divisor) {
    const uint32_t lane = lane_id(), wave = threadIdx.x / kWave;
    uint2 before = make_uint2(0u, 0u);                       // lane u: of wave u, if it comes before this one
    if (lane < wave) before = counts[lane];
    uint32_t out = few_lanes_sum(before.x), eq = 0;
    if (!PLAIN) {
        eq = few_lanes_sum(before.y);
        out += (eq < c.ties ? eq : c.ties) - eq;
    }
    out = (uint32_t)__builtin_amdgcn_readfirstlane((int)(out + c.out));
    const uint32_t least = once_more(c.least);
    uint32_t lo = 0, hi = 0;                                 // the masks
    const uint2 mine = counts[wave];
    if (out + mine.x > k + mine.y) return 0ull;              // (never when the state is consistent)
    uint32_t* oi = out_idx + out;
    uint32_t* ov = reinterpret_cast<uint32_t*>(out_val) + out;
    uint32_t run = 0;                                        // selected in the steps before
    uint32_t index = first_index + lane;
    asm volatile("" : "+v"(index));                          // (else sixteen sums of it are kept from side to side)
    for_live_steps(once_more(live), [&](auto step) {
        constexpr int j = decltype(step)::j;
        bool sel = reaches<PLAIN>(v[j], least);
        if (!PLAIN && c.ranked) {                            // block-uniform
            const bool is_eq = (v[j] & kAbs) == least;
            const uint64_t eqm = __ballot(is_eq);
            sel = sel && (!is_eq || eq + rank_in(eqm) < c.ties);
            eq += (uint32_t)__popcll(eqm);
        }
        const uint64_t m = __ballot(sel);
        set_lane<j>(lo, hi, m);
        if (sel) {
            const uint32_t pos = rank_from(m, run);
            if (PLAIN || out + pos < k) {                    // (likewise)
                store_at(oi, pos, index + j * kWave);
                const float x = __uint_as_float(v[j]);
                store_at(ov, pos, __float_as_uint(DIVIDE ? x / divisor : x));
            }
        }
        v[j] = sel ? v[j] : kNone<PLAIN>;
        run += (uint32_t)__popcll(m);
    });
    return (uint64_t)lo | (uint64_t)hi << 32;
}

// What a block leaves for the select of the next round's pair: the sum of its two sides, in registers.
struct GroupNext {
    uint32_t first;             // number of the first pair
    float* keys;                // [pairs][key_stride] bracket keys
    size_t key_stride;
    uint32_t* samples;          // [pairs][ngroups * per_group] or NULL
    uint32_t per_group;
};
// a becomes the union of a and b; s_hist: kBrkBins / 2 words of LDS, zero; s_in: a word per wave.  region: the two sides'
// first output positions together, where the group's keys go (a union holds no more entries than its operands).
template <bool PLAIN>
__device__ __forceinline__ void count_union(uint32_t (&a)[kGrpPer], const uint32_t (&b)[kGrpPer], uint32_t live, const GroupSets& gs,
                                            const GroupNext& nx, const Bracket& bk, uint32_t p, uint32_t g, uint32_t region,
                                            uint32_t* s_hist, uint32_t* s_in) {
    const uint32_t lane = lane_id(), wave = threadIdx.x / kWave;
    const uint32_t id = nx.first + p;
    uint32_t in = 0, above = 0;                              // wave-uniform
    uint64_t any[4] = {0ull, 0ull, 0ull, 0ull};
    for_live_steps(once_more(live), [&](auto step) {
        constexpr int j = decltype(step)::j;
        a[j] = sum_of<PLAIN>(a[j], b[j]);
        const uint64_t up = __ballot(reaches<PLAIN>(a[j], bk.hi));
        const uint64_t m = __ballot(reaches<PLAIN>(a[j], bk.lo)) & ~up;
        above += (uint32_t)__popcll(up);
        in += (uint32_t)__popcll(m);
        any[j / 4] |= m;
    });
    const uint32_t hit = (any[0] ? 1u : 0u) | (any[1] ? 2u : 0u) | (any[2] ? 4u : 0u) | (any[3] ? 8u : 0u);
    if (nx.samples) {
        const uint32_t h = sample_hash(g, wave), at = sample_step(h), q = nx.per_group / kGrpWaves;
        uint32_t v = kNone<PLAIN>;
        for_live_steps(once_more(live), [&](auto step) {
            constexpr int j = decltype(step)::j;
            if ((uint32_t)j == at) v = a[j];
        });
        v = __shfl(v, sample_lane(h, lane, q));
        if (lane < q) nx.samples[((size_t)p * gs.ngroups + g) * nx.per_group + wave * q + lane] = v;
    }
    if (lane == 0) s_in[wave] = in | above << 16;            // (at most 1024 of a wave)
    __syncthreads();
    const uint32_t all = lane < (uint32_t)kGrpWaves ? s_in[lane] : 0u;
    uint32_t off = few_lanes_sum(lane < wave ? all & 0xFFFFu : 0u);
    const uint32_t both = few_lanes_sum(all), all_in = both & 0xFFFFu, all_above = both >> 16;
    if (threadIdx.x == 0) gs.run[(size_t)id * gs.ngroups + g] = make_uint4(region, all_in, all_above, kPlainRun);
    off = (uint32_t)__builtin_amdgcn_readfirstlane((int)(off + region));
    if (in && off + in <= nx.key_stride) {                   // (the second is always so)
        uint32_t* keys = reinterpret_cast<uint32_t*>(nx.keys) + (size_t)p * nx.key_stride + off;
        const uint32_t lo = once_more(bk.lo), width = once_more(bk.hi) - lo;
        uint32_t run = 0;
        for_live_steps(once_more(hit), [&](auto step) {
            constexpr int j = decltype(step)::j;
            const uint32_t rel = (a[j] & kAbs) - lo;         // (the key of kAbsent is above any bracket)
            const bool is_in = rel < width;
            const uint64_t m = __ballot(is_in);
            if (is_in) {
                store_at(keys, rank_from(m, run), rel + lo);
                atomicAdd(&s_hist[rel >> bk.shift], 1u);
            }
            run += (uint32_t)__popcll(m);
        });
    }
    __syncthreads();
    uint32_t* out = gs.hist + (size_t)id * kBrkBins;
    for (uint32_t w = threadIdx.x; w < (uint32_t)kBrkBins / 2; w += kGrpBlock) {
        const uint32_t c = s_hist[w];
        if (c) atomicAdd(&out[w], c);
    }
    if (threadIdx.x == 0 && all_above) atomicAdd(&out[kAboveBin], all_above);
}
// the same for a group without any entry
__device__ __forceinline__ void count_nothing(const GroupSets& gs, const GroupNext& nx, uint32_t p, uint32_t g, uint32_t region) {
    if (threadIdx.x == 0) gs.run[(size_t)(nx.first + p) * gs.ngroups + g] = make_uint4(region, 0u, 0u, kPlainRun);
    if (nx.samples && threadIdx.x < nx.per_group)
        nx.samples[((size_t)p * gs.ngroups + g) * nx.per_group + threadIdx.x] = kAbsent;
}

struct GroupShared {
    uint32_t hist[kBrkBins / 2];
    uint2 cnt[2][kGrpWaves];
    uint32_t in[kGrpWaves];
};
constexpr uint32_t kGroupWords = kGroup / 64;                // words of a bit per element

template <bool PLAIN>
__device__ __forceinline__ void select_pair(GroupShared& sh, const GroupSets& gs, const GroupNext& nx, const Bracket& bk,
                                            const GroupCut (&cut)[2], const uint64_t (&mask)[2], const float* __restrict__ rows,
                                            int64_t stride, uint32_t k, uint32_t* __restrict__ out_idx,
                                            float* __restrict__ out_val, uint64_t* __restrict__ bits) {
    const uint32_t g = blockIdx.x, p = blockIdx.y;
    const uint32_t lane = lane_id(), wave = threadIdx.x / kWave;
    // (uniform across the wave: the loads share one address and differ by constants)
    const uint32_t first = (uint32_t)__builtin_amdgcn_readfirstlane((int)(g * kGroup + wave * (kGrpPer * kWave)));
    const uint32_t left = first < gs.m ? gs.m - first : 0u;
    uint32_t v[2][kGrpPer], live[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const float* row = rows + (int64_t)(2u * p + s) * stride + first;
        live[s] = (uint32_t)__builtin_amdgcn_readfirstlane((int)((uint32_t)(mask[s] >> (wave * 4u)) & 15u));
#pragma unroll
        for (int b = 0; b < kGrpPer / 4; ++b) {
#pragma unroll
            for (int j = 4 * b; j < 4 * b + 4; ++j) v[s][j] = kNone<PLAIN>;
            if (((live[s] >> b) & 1u) == 0u) continue;
            if ((uint32_t)(4 * b + 4) * kWave <= left) {
#pragma unroll
                for (int j = 4 * b; j < 4 * b + 4; ++j) v[s][j] = kept<PLAIN>(__float_as_uint(row[j * kWave + lane]));
            } else {
#pragma unroll
                for (int j = 4 * b; j < 4 * b + 4; ++j)
                    if (j * kWave + lane < left) v[s][j] = kept<PLAIN>(__float_as_uint(row[j * kWave + lane]));
            }
        }
    }
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const uint2 c = count_cut<PLAIN>(v[s], live[s], cut[s]);
        if (lane == 0) sh.cnt[s][wave] = c;
    }
    __syncthreads();
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const uint32_t w = 2u * p + s;
        const uint64_t b = emit_cut<PLAIN, false>(v[s], live[s], cut[s], sh.cnt[s], first, k, out_idx + (size_t)w * k,
                                                  out_val + (size_t)w * k, 1.0f);
        if (lane < (uint32_t)kGrpPer) bits[((size_t)w * gs.ngroups + g) * kGroupWords + wave * kGrpPer + lane] = b;
    }
    count_union<PLAIN>(v[0], v[1], live[0] | live[1], gs, nx, bk, p, g, cut[0].out + cut[1].out, sh.hist, sh.in);
}

// Block (g, p): group g of workers 2p and 2p + 1.  Only the stretches that hold candidates are read.  bits: one bit per
// element of a row, the worker's set (for the restore).
// Bound by instruction issue as much as by memory (some 70 vector and 60 scalar instructions per 64 elements of the pair before
// keys were compared as numbers and steps without candidates skipped, half of that now): 880 us for 4.2 GB (by the counters) =
// 4.8 TB/s at m = 25,557,032, P = 32, k = 6.4 M; 720 us where fewer stretches hold candidates.  64 registers, so that four blocks share a CU: with spills 803 us.
__global__ __launch_bounds__(kGrpBlock) __attribute__((amdgpu_waves_per_eu(8, 8))) void k_group_select(
        GroupSets gs, GroupNext nx, const float* __restrict__ rows, int64_t stride, uint32_t k, uint32_t* __restrict__ out_idx,
        float* __restrict__ out_val, uint64_t* __restrict__ bits) {
    __shared__ GroupShared sh;
    const uint32_t g = blockIdx.x, p = blockIdx.y;
    GroupCut cut[2];
    uint64_t mask[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const uint32_t w = 2u * p + s, head = (uint32_t)(((int64_t)w * stride) & 3);
        cut[s] = group_cut(gs, w, g);
        const uint64_t* mk = gs.mask + (size_t)w * (gs.ngroups + 1u) + g;
        uint64_t x = mk[0];
        if (head) {                                          // stretches are cut on v = index + head
            x |= x >> 1;
            if (((uint64_t)(g + 1u) << kGroupLog2) < (uint64_t)gs.m + head) x |= mk[1] << (kGroup / 256u - 1u);
        }
        mask[s] = gs.T[w] < gs.lo[w] ? ~0ull : x;            // (a set that missed its bracket: entries anywhere)
    }
    if ((mask[0] | mask[1]) == 0u) {                         // block-uniform
        count_nothing(gs, nx, p, g, cut[0].out + cut[1].out);
        if (threadIdx.x < 2 * kGroupWords)
            bits[((size_t)(2u * p + threadIdx.x / kGroupWords) * gs.ngroups + g) * kGroupWords + threadIdx.x % kGroupWords] = 0ull;
        return;
    }
    for (uint32_t b = threadIdx.x; b < (uint32_t)kBrkBins / 2; b += kGrpBlock) sh.hist[b] = 0u;     // a barrier follows
    const Bracket bk(gs, nx.first + p);
    if (plain_cut(cut[0]) && plain_cut(cut[1]) && bk.lo != 0u)       // block-uniform
        select_pair<true>(sh, gs, nx, bk, cut, mask, rows, stride, k, out_idx, out_val, bits);
    else
        select_pair<false>(sh, gs, nx, bk, cut, mask, rows, stride, k, out_idx, out_val, bits);
}

template <int SIDES, bool PLAIN>
__device__ __forceinline__ void merge_pairs(GroupShared& sh, uint32_t* s_cell, const GroupSets& gs, const GroupNext& nx,
                                            const Bracket& bk, const Operands (&o)[SIDES], const GroupCut (&cut)[SIDES], uint32_t k,
                                            uint32_t* __restrict__ out_idx, float* __restrict__ out_val, float divisor,
                                            uint64_t* __restrict__ gbits) {
    const uint32_t g = blockIdx.x, p = blockIdx.y;
    const uint32_t lane = lane_id(), wave = threadIdx.x / kWave;
    const uint32_t first = g * kGroup + wave * (kGrpPer * kWave);
    uint32_t v[SIDES][kGrpPer], live[SIDES];
    OperandBatch b[SIDES];                                   // (all sides' first loads in flight together)
#pragma unroll
    for (int s = 0; s < SIDES; ++s)
#pragma unroll
        for (int j = 0; j < 2; ++j) load_operand(o[s], j, o[s].first[j], b[s].idx[j], b[s].val[j]);
    clear_cells<PLAIN>(s_cell);
#pragma unroll
    for (int s = 0; s < SIDES; ++s) {
        unite<PLAIN>(o[s], b[s], g, s_cell);
        uint32_t* own = s_cell + wave * (kGrpPer * kWave) + lane;
#pragma unroll
        for (int j = 0; j < kGrpPer; ++j) {
            v[s][j] = own[j * kWave];
            if (s + 1 < SIDES) own[j * kWave] = kNone<PLAIN>;        // (for the next side)
        }
        live[s] = 0;
#pragma unroll
        for (int q = 0; q < kGrpPer / 4; ++q)
            live[s] |= __any(v[s][4 * q] != kNone<PLAIN> || v[s][4 * q + 1] != kNone<PLAIN> || v[s][4 * q + 2] != kNone<PLAIN> ||
                             v[s][4 * q + 3] != kNone<PLAIN>) ? 1u << q : 0u;
        const uint2 c = count_cut<PLAIN>(v[s], live[s], cut[s]);
        if (lane == 0) sh.cnt[s][wave] = c;
        __syncthreads();
        const size_t row = (size_t)(SIDES * p + s) * k;
        const uint64_t bits = emit_cut<PLAIN, SIDES == 1>(v[s], live[s], cut[s], sh.cnt[s], first, k, out_idx + row, out_val + row, divisor);
        if (SIDES == 1 && lane < (uint32_t)kGrpPer) gbits[(size_t)g * kGroupWords + wave * kGrpPer + lane] = bits;
    }
    if constexpr (SIDES == 2)
        count_union<PLAIN>(v[0], v[1], live[0] | live[1], gs, nx, bk, p, g, cut[0].out + cut[1].out, sh.hist, sh.in);
}

// Bound like the select: 539 us for the 2.5 GB of the first of these rounds at the same size, each further one half of that.
// Groups of 8192 and blocks of 512 threads: 603 / 340 us at k = 6.4 M / 1.85 M against 651 / 377 with twice that.  Four entries of
// each operand ahead per thread: eight spill (707 us), all sides' first entries loaded together 534 -> 539 us, but fewer barriers.
// SIDES == 2: block (g, p) forms group g of pairs 2p and 2p + 1 of this round (numbers first_pair + ..), emits their
// selected entries and counts the union of the two for the next round.  SIDES == 1, the last round: the pair's entries
// are divided by `divisor` (Eq. 3) and the global set's bits stored (all words).
template <int SIDES>
__global__ __launch_bounds__(kGrpBlock) __attribute__((amdgpu_waves_per_eu(8, 8))) void k_group_merge(
        GroupSets gs, GroupNext nx, uint32_t first_pair, uint32_t first_in, const uint32_t* __restrict__ in_idx,
        const float* __restrict__ in_val, uint32_t k, uint32_t* __restrict__ out_idx, float* __restrict__ out_val, float divisor,
        uint64_t* __restrict__ gbits) {
    __shared__ uint32_t s_cell[kGroup];
    __shared__ GroupShared sh;
    const uint32_t g = blockIdx.x, p = blockIdx.y;
    Operands o[SIDES];
    GroupCut cut[SIDES];
    uint32_t entries = 0, region = 0;
    bool plain = true;
#pragma unroll
    for (int s = 0; s < SIDES; ++s) {
        o[s] = group_operands(gs, in_idx, in_val, first_in, k, SIDES * p + s, g);
        entries += o[s].end[0] - o[s].first[0] + o[s].end[1] - o[s].first[1];
        cut[s] = group_cut(gs, first_pair + SIDES * p + s, g);
        region += cut[s].out;
        plain = plain && plain_cut(cut[s]);
    }
    if (entries == 0u) {                                     // block-uniform
        if (SIDES == 2) count_nothing(gs, nx, p, g, region);
        else if (threadIdx.x < kGroupWords) gbits[(size_t)g * kGroupWords + threadIdx.x] = 0ull;
        return;
    }
    if (SIDES == 2)
        for (uint32_t b = threadIdx.x; b < (uint32_t)kBrkBins / 2; b += kGrpBlock) sh.hist[b] = 0u;
    const Bracket bk(gs, SIDES == 2 ? nx.first + p : first_pair);
    if (plain && (SIDES == 1 || bk.lo != 0u))                // block-uniform
        merge_pairs<SIDES, true>(sh, s_cell, gs, nx, bk, o, cut, k, out_idx, out_val, divisor, gbits);
    else
        merge_pairs<SIDES, false>(sh, s_cell, gs, nx, bk, o, cut, k, out_idx, out_val, divisor, gbits);
}

// ---------------------------------------------------------------------------------
// residual restore (Algorithm 4 line 10), fused form: see k_restore_fused
// ---------------------------------------------------------------------------------

// A slot whose index is in the worker's set and in the global one becomes +0.0, and one that holds a selected -0.0
// (only in a set that reaches down to key 0).  Lane = element, a wave's stores fall into whole lines where the sets
// are dense; bound by partial lines, which memory reads before it writes them: words with many slots to clear are read and
// written whole, from 16 of 64 on.  us with words whole from 1 / 4 / 8 / 16 on / never, m = 25,557,032, P = 32, layers: k = 6.4 M
// 729 / 788 / 797 / 790 / 820, k = 1.85 M 538 / 413 / 370 / 343 / 346 (and a row without layers loses 900 us at k = m / 8 with 1).
constexpr uint32_t kRestoreWhole = 16;
constexpr int kRestoreWords = 16;                            // per wave: as many loads are in flight
__global__ __launch_bounds__(kBlock) void k_group_restore(
        float* __restrict__ res, int64_t stride, GroupSets gs, const uint64_t* __restrict__ bits, const uint64_t* __restrict__ gbits) {
    const uint32_t w = blockIdx.y, lane = lane_id();
    const uint32_t words = gs.ngroups * kGroupWords;         // a multiple of kRestoreWords
    const uint32_t word0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)((blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave) * kRestoreWords));
    if (word0 >= words) return;
    uint64_t mine = 0, both = 0;
    if (lane < (uint32_t)kRestoreWords) {
        mine = bits[(size_t)w * words + word0 + lane];
        both = mine & gbits[word0 + lane];
    }
    float* row = res + (int64_t)w * stride + (size_t)word0 * 64u;
    auto word = [&](uint64_t x, int u) {
        return (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, u) |
               (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(x >> 32), u) << 32;
    };
    if (gs.T[w] == 0u) {                                     // block-uniform
        for (int u = 0; u < kRestoreWords; ++u) {
            const bool in = (word(mine, u) >> lane) & 1u, clear = (word(both, u) >> lane) & 1u;
            if (clear || (in && __float_as_uint(row[u * 64 + lane]) == 0x80000000u)) row[u * 64 + lane] = 0.0f;
        }
        return;
    }
    // words with kRestoreWhole slots to clear, or more, are read and written back as whole lines, the others' slots stored alone
    const uint32_t some = (uint32_t)__ballot(both != 0ull);
    const uint32_t whole = (uint32_t)__ballot((uint32_t)__popcll(both) >= kRestoreWhole && (word0 + lane + 1u) * 64u <= gs.m);
    if (some == 0u) return;
    float x[kRestoreWords];
#pragma unroll
    for (int u = 0; u < kRestoreWords; ++u)
        if ((whole >> u) & 1u) x[u] = __builtin_nontemporal_load(row + u * 64 + lane);
#pragma unroll
    for (int u = 0; u < kRestoreWords; ++u) {
        if (((some >> u) & 1u) == 0u) continue;
        const bool clear = (word(both, u) >> lane) & 1u;
        if ((whole >> u) & 1u) __builtin_nontemporal_store(clear ? 0.0f : x[u], row + u * 64 + lane);
        else if (clear) row[u * 64 + lane] = 0.0f;
    }
}

}  // namespace gtopk
