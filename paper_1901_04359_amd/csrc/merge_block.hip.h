// The Top-k operation between two sparse vectors (Definition 1) of up to kMergeBlockMaxK entries each: one block
// does all of it - union, exact select, ordered emit - with both operands in LDS and the merged slots in registers.
// For sets of this size the three kernels of the general path (union, walk, emit) are bound by launch and drain and by
// what every one of their blocks repeats, not by bytes (a round of sets of 1000 entries 19.5 us, here 9.5; of 8192 entries
// 20.5 / 20).  Here the per-thread chain bounds: about 0.8 us per slot of a thread on top of some 8 us.
#pragma once
#include "common.hip.h"

namespace gtopk {

constexpr int kMbBlock = 1024;
constexpr uint32_t kMergeBlockMaxK = 8192;

// Thread t owns the EPT slots from t * EPT on of the union in index order (2k slots, A's copy of a shared index first,
// with the sum; B's copy is a tombstone): it finds its place by a binary search along the diagonal and merges EPT steps.
// Keys stay in registers from there on: the first digit of all of them and the lower digits of those in the k-th key's
// bin are counted in LDS, one block scan gives every thread its output positions, and the selected entries leave
// through LDS in whole rows.  k <= kMbBlock / 2 * EPT.
// in_min: smallest keys of the operands (2 per pair), NULL: found here.  inverted: see MergedSrc.
// Slots past either operand's end are spare (EPT of them): with operands that are not sorted (unspecified results) a
// thread may run that far.
template <int EPT, bool DIVIDE>
__global__ __launch_bounds__(kMbBlock) void k_merge_block(
        const uint32_t* __restrict__ a_idx, const float* __restrict__ a_val, const uint32_t* __restrict__ b_idx,
        const float* __restrict__ b_val, uint32_t k, int64_t in_stride, uint32_t* __restrict__ out_idx,
        float* __restrict__ out_val, int64_t out_stride, const uint32_t* __restrict__ in_min, bool inverted,
        uint32_t* __restrict__ out_min, float divisor, uint32_t* __restrict__ gbits) {
    constexpr uint32_t kCap = kMbBlock / 2 * EPT;            // entries per operand, at most
    constexpr uint32_t kRow = kCap + EPT + 1;
    constexpr int kShare = (EPT + 1) / 2;                    // entries of either operand that a thread loads
    __shared__ uint32_t s_i[2 * kRow];
    __shared__ uint32_t s_v[2 * kRow];
    __shared__ uint32_t s_h[kHistBins];
    __shared__ uint32_t s_wave[kMbBlock / kWave];
    __shared__ uint32_t s_out[3];
    __shared__ uint32_t s_min[2];
    const uint32_t t = threadIdx.x;
    const int s = blockIdx.x;
    const uint32_t* ai = a_idx + (int64_t)s * in_stride;
    const uint32_t* bi = b_idx + (int64_t)s * in_stride;
    const uint32_t* av = reinterpret_cast<const uint32_t*>(a_val) + (int64_t)s * in_stride;
    const uint32_t* bv = reinterpret_cast<const uint32_t*>(b_val) + (int64_t)s * in_stride;
    uint32_t va[kShare], vb[kShare];
    {
        uint32_t ia[kShare], ib[kShare];
#pragma unroll
        for (int r = 0; r < kShare; ++r) {
            const uint32_t i = r * kMbBlock + t;
            const bool live = i < k;
            ia[r] = live ? ai[i] : kTomb;
            ib[r] = live ? bi[i] : kTomb;
            va[r] = live ? av[i] : kAbs;                     // the largest key: changes no minimum
            vb[r] = live ? bv[i] : kAbs;
        }
        if (t < 2) s_min[t] = 0u;
        for (uint32_t b = t; b < (uint32_t)kHistBins; b += kMbBlock) s_h[b] = 0u;
#pragma unroll
        for (int r = 0; r < kShare; ++r) {
            const uint32_t i = r * kMbBlock + t;
            if (i < kCap) {
                s_i[i] = ia[r];
                s_i[kRow + i] = ib[r];
                s_v[i] = va[r];
                s_v[kRow + i] = vb[r];
            }
        }
        if (t <= (uint32_t)EPT) s_i[kCap + t] = s_i[kRow + kCap + t] = kTomb;
    }
    __syncthreads();
    if (!in_min) {
        uint32_t ma = 0, mb = 0;                             // kAbs - smallest key
#pragma unroll
        for (int r = 0; r < kShare; ++r) {
            const uint32_t x = kAbs - (va[r] & kAbs), y = kAbs - (vb[r] & kAbs);
            ma = x > ma ? x : ma;
            mb = y > mb ? y : mb;
        }
        ma = wave_largest(ma);
        mb = wave_largest(mb);
        if (lane_id() == 0) {
            atomicMax(&s_min[0], ma);
            atomicMax(&s_min[1], mb);
        }
        __syncthreads();
    }
    uint32_t lo_a = in_min ? in_min[2 * s] : s_min[0], lo_b = in_min ? in_min[2 * s + 1] : s_min[1];
    if (!in_min || inverted) {
        lo_a = kAbs - lo_a;
        lo_b = kAbs - lo_b;
    }
    const Digit dg{lo_a > lo_b ? lo_a : lo_b, (uint32_t)kFineShift};

    // ---- union --------------------------------------------------------------------------
    const uint32_t* sa = s_i;
    const uint32_t* sb = s_i + kRow;
    const uint32_t d = t * EPT, n = 2 * k;
    uint32_t oi[EPT], ov[EPT];
#pragma unroll
    for (int j = 0; j < EPT; ++j) { oi[j] = kTomb; ov[j] = 0u; }
    if (d < n) {
        uint32_t x = d > k ? d - k : 0u, hi = d < k ? d : k;
        while (x < hi) {
            const uint32_t mid = (x + hi) >> 1;
            if (sa[mid] <= sb[d - 1 - mid]) x = mid + 1; else hi = mid;
        }
        uint32_t y = d - x;
        uint32_t a = sa[x], b = sb[y], aprev = x > 0 ? sa[x - 1] : kTomb;
#pragma unroll
        for (int j = 0; j < EPT; ++j) {
            if (d + j >= n) continue;
            if (a <= b) {
                oi[j] = a;
                ov[j] = s_v[x];
                if (b == a) ov[j] = __float_as_uint(__uint_as_float(ov[j]) + __uint_as_float(s_v[kRow + y]));
                aprev = a;
                a = sa[++x];
            } else {
                const bool dup = b == aprev;
                oi[j] = dup ? kTomb : b;
                ov[j] = s_v[kRow + y];
                b = sb[++y];
            }
        }
    }
    // ---- the k-th key ---------------------------------------------------------------------
#pragma unroll
    for (int j = 0; j < EPT; ++j)
        if (oi[j] != kTomb) atomicAdd(&s_h[dg.bin(ov[j] & kAbs)], 1u);
    __syncthreads();
    uint32_t krem = k, base, width;
    {
        constexpr int kPer = kHistBins / kMbBlock;
        uint32_t loc[kPer];
#pragma unroll
        for (int j = 0; j < kPer; ++j) loc[j] = s_h[t * kPer + j];
        suffix_pick<kPer>(loc, k, s_wave, s_out);
        krem -= s_out[1];
        base = dg.lo(s_out[0]);
        width = dg.width(s_out[0]);
    }
    // lower digits of the keys in its bin: bits 30..20, 19..10, 9..0 of key - base; a pass whose bits are zero for the
    // whole bin is skipped
    uint32_t prefix = 0;
    for (int pass = 0; pass < 3; ++pass) {
        const int shift = pass == 0 ? 20 : (pass == 1 ? 10 : 0);
        const int bits = pass == 0 ? 11 : 10;
        if (shift > 0 && width <= (1u << shift)) continue;   // uniform
        __syncthreads();                                     // s_h and s_out have been read
        s_h[t] = 0u;
        s_h[t + kMbBlock] = 0u;
        __syncthreads();
#pragma unroll
        for (int j = 0; j < EPT; ++j) {
            const uint32_t rel = (ov[j] & kAbs) - base;
            if (oi[j] != kTomb && rel < width && (rel >> (shift + bits)) == prefix)
                atomicAdd(&s_h[(rel >> shift) & ((1u << bits) - 1u)], 1u);
        }
        __syncthreads();
        const uint32_t loc[2] = {s_h[2 * t], s_h[2 * t + 1]};
        suffix_pick<2>(loc, krem, s_wave, s_out);
        prefix = (prefix << bits) | s_out[0];
        krem -= s_out[1];
    }
    const uint32_t T = base + prefix, need = krem;

    // ---- emit -----------------------------------------------------------------------------
    uint32_t mine = 0;                                       // entries above T, and equal to it << 16
#pragma unroll
    for (int j = 0; j < EPT; ++j) {
        const uint32_t key = ov[j] & kAbs;
        if (oi[j] != kTomb) mine += key > T ? 1u : (key == T ? 0x10000u : 0u);
    }
    uint32_t total;
    const uint32_t before = block_incl_scan(mine, s_wave, total) - mine;
    uint32_t eq = before >> 16, pos = (before & 0xFFFFu) + (eq < need ? eq : need);
    static_assert(kMergeBlockMaxK < 65536u, "16-bit counts: fewer than k above T, at most 2k equal to it");
    uint32_t* so_i = s_i;                                    // (every thread is behind its last use of the operands)
    uint32_t* so_v = s_i + kRow;
#pragma unroll
    for (int j = 0; j < EPT; ++j) {
        if (oi[j] == kTomb) continue;
        const uint32_t key = ov[j] & kAbs;
        bool sel = key > T;
        if (key == T) sel = eq++ < need;
        if (sel && pos < kCap) {                             // (always so)
            so_i[pos] = oi[j];
            so_v[pos] = ov[j];
            ++pos;
        }
    }
    __syncthreads();
    uint32_t* oi_row = out_idx + (int64_t)s * out_stride;
    float* ov_row = out_val + (int64_t)s * out_stride;
    const uint32_t eqs = total >> 16, kept = (total & 0xFFFFu) + (eqs < need ? eqs : need);
    const uint32_t count = kept < k ? kept : k;              // (k, unless an operand holds an index twice)
    for (uint32_t i = t; i < count; i += kMbBlock) {
        const uint32_t ix = so_i[i];
        const float v = __uint_as_float(so_v[i]);
        oi_row[i] = ix;
        ov_row[i] = DIVIDE ? v / divisor : v;
        // the first entry of each run that shares a bitmap word sets the bits of the whole run
        if (gbits && (i == 0 || (so_i[i - 1] >> 5) != (ix >> 5))) {
            uint32_t bits = 1u << (ix & 31);
            for (uint32_t q = i + 1; q < count && (so_i[q] >> 5) == (ix >> 5); ++q) bits |= 1u << (so_i[q] & 31);
            atomicOr(&gbits[ix >> 5], bits);
        }
    }
    if (t == 0 && out_min) out_min[s] = T;
}

}  // namespace gtopk
