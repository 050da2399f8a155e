// The hot path for small problems (short rows, few workers, few selected entries), where a
// step is bound by the number of dependent kernel launches and not by bytes:
//   k_small_sample  the speculative threshold of one worker in ONE block (sample histogram
//                   in LDS and the pick), which also clears the worker's candidate counter;
//   k_small_select  the exact local selection (Algorithm 4 lines 5-7) of one worker in ONE
//                   block, with block-level synchronisation only: a short candidate list
//                   in registers, anything else by histogram, radix refinement and ordered emit;
//   k_small_tree    the whole gTopKAllReduce tree (Algorithm 3 lines 4-18: every round's
//                   Top-k operations of Definition 1), the division by P (Eq. 3) and the
//                   extra residual (Algorithm 4 line 10) in ONE block, all sets in LDS.
// The last two produce bit for bit what the general kernels produce; the threshold of the
// first only sizes the work.
#pragma once
#include "common.hip.h"
#include "select.hip.h"

namespace gtopk {

constexpr int kSmallBlock = 1024;
constexpr int kSmallIters = 2;               // float4 per lane of the streaming pass's blocks
constexpr int kSmallChunk = kSmallIters * 4 * kSBlock;      // 4096 elements per block = one run
constexpr int kSmallMaxChunks = 256;         // rows of at most 2^20 elements
constexpr int kSmallMaxEntries = 4096;       // P * k, at most
constexpr int kSmallMaxK = 512;
constexpr int kSmallMaxP = 64;
constexpr int kSmallEntries = 2;             // entries per thread of a candidate list held in registers
constexpr int kMidSampleTile = 16;           // elements per tile where it serves rows of millions of elements
constexpr int kRowPart = 16;                 // entries per thread where the parts of a row come together
constexpr int kSmallSampleUnroll = 16;       // tiles that each of its groups of lanes keeps in flight

__device__ __forceinline__ uint32_t op_max(uint32_t a, uint32_t b) { return a > b ? a : b; }

// ---------------------------------------------------------------------------------
// selection by a team of waves
// ---------------------------------------------------------------------------------

constexpr int kTreeEpt = kSmallMaxEntries / kSmallBlock;
constexpr int kTreeTeams = 8;
constexpr uint32_t kTreeBins = 1024;
constexpr uint32_t kTreeList = 32;
// bin of a key at distance rel from the bound: the distance itself below 32, then 32 bins per octave
__device__ __forceinline__ uint32_t tree_bin(uint32_t rel) {
    if (rel < 32u) return rel;
    const uint32_t e = 31u - (uint32_t)__builtin_clz(rel);
    return ((e - 4u) << 5) + ((rel >> (e - 5u)) & 31u);
}
// smallest distance of bin b, and how many distances it holds (as a power of two)
__device__ __forceinline__ uint32_t tree_bin_first(uint32_t b) { return b < 32u ? b : (32u + (b & 31u)) << ((b >> 5) - 1u); }
__device__ __forceinline__ uint32_t tree_bin_bits(uint32_t b) { return b < 32u ? 0u : (b >> 5) - 1u; }


template <int TEAMS>
struct TeamShared {
    __align__(16) uint32_t hist[TEAMS * kTreeBins];            // zero between selections
    uint32_t list[TEAMS][kTreeList];
    uint32_t wave[kSmallBlock / kWave];
    uint32_t pick[TEAMS][3], n[TEAMS], T[TEAMS], need[TEAMS];
};
template <int TEAMS>
__device__ __forceinline__ void clear_teams(TeamShared<TEAMS>& sh) {
    for (uint32_t b = 4 * threadIdx.x; b < TEAMS * kTreeBins; b += 4 * kSmallBlock)
        *reinterpret_cast<uint4*>(&sh.hist[b]) = make_uint4(0u, 0u, 0u, 0u);
}

// Each of the block's teams of SIZE threads (>= a wave) selects the k largest of its threads' keys (E each, kNoKey:
// none), among equal ones the first in thread order.  The keys from `bound` on, which k of them are expected to reach,
// are counted in 1024 bins that widen with the distance (a 32nd of an octave each), the team picks the bin of the k-th, and
// while that holds more than kTreeList keys it is cut into 1024 again; what is left goes to a list, where every key's
// owner ranks it.  Every thread of the block calls it; about eight barriers.
struct TeamCut { uint32_t T, need, pos, eq; };     // the k-th key, keys equal to it to take; selected before this thread, equal ones before it
template <uint32_t SIZE, int TEAMS, int E>
__device__ __forceinline__ TeamCut team_select(TeamShared<TEAMS>& sh, const uint32_t (&key)[E], uint32_t bound, uint32_t k) {
    constexpr uint32_t team_waves = SIZE / kWave, per = kTreeBins / SIZE;      // bins per thread
    const uint32_t t = threadIdx.x, lane = lane_id(), wave = t / kWave;
    const uint32_t team = t / SIZE, l = t % SIZE, first_wave = team * team_waves;
    uint32_t* hist = sh.hist + team * kTreeBins;
    // the k-th key lies in base + [lo, lo + 2^bits), `rank` of the `count` keys there reach it.  base: the bound,
    // which k keys of the union reach unless sums cancel, else 0.
    uint32_t base = bound, lo = 0, bits = 31, rank = k, count = 0;
    bool by_octave = true, more = true;
    auto candidate = [&](int j) {
        return key[j] >= base && key[j] - base - lo < (1u << bits);            // (never kNoKey)
    };
    do {                                       // (every thread of the block takes the same turns)
        const uint32_t shift = bits > 10u ? bits - 10u : 0u;
        if (more)
#pragma unroll
            for (int j = 0; j < E; ++j)
                if (candidate(j)) {
                    const uint32_t rel = key[j] - base;
                    atomicAdd(&hist[by_octave ? tree_bin(rel) : (rel - lo) >> shift], 1u);
                }
        __syncthreads();
        uint32_t mine = 0, loc[per];
#pragma unroll
        for (uint32_t i = 0; i < per; ++i) {
            loc[i] = hist[l * per + i];
            hist[l * per + i] = 0u;            // (for the next turn, and the next round)
            mine += loc[i];
        }
        const uint32_t incl = wave_incl_scan(mine);
        if (lane == kWave - 1) sh.wave[wave] = incl;
        if (l == 0) { sh.pick[team][2] = 0u; sh.n[team] = 0u; }
        __syncthreads();
        const uint32_t sums = row_incl_scan(lane < team_waves ? sh.wave[first_wave + lane] : 0u);
        const uint32_t w_in = wave - first_wave;
        uint32_t above = lane_value(sums, 15u) - incl - (w_in ? lane_value(sums, w_in - 1u) : 0u);
        if (above < rank && above + mine >= rank) {                     // one thread owns the crossing
#pragma unroll
            for (int i = (int)per - 1; i >= 0; --i) {
                if (above < rank && above + loc[i] >= rank) {
                    sh.pick[team][0] = l * per + (uint32_t)i;
                    sh.pick[team][1] = above;
                    sh.pick[team][2] = loc[i];
                }
                above += loc[i];
            }
        }
        __syncthreads();
        if (more) {
            const uint32_t b = sh.pick[team][0], c = sh.pick[team][2];
            if (c == 0u) {                     // fewer than k keys reach the bound
                more = base != 0u;             // (always so: the union has k entries)
                if (!more) bits = 0;
                base = 0;
            } else {
                rank -= sh.pick[team][1];
                count = c;
                lo = by_octave ? tree_bin_first(b) : lo + (b << shift);
                bits = by_octave ? tree_bin_bits(b) : shift;
                by_octave = false;
                more = count > kTreeList && bits > 0u;
            }
        }
    } while (__syncthreads_or(more ? 1 : 0));
    if (bits > 0u) {
#pragma unroll
        for (int j = 0; j < E; ++j)
            if (candidate(j)) sh.list[team][atomicAdd(&sh.n[team], 1u) & (kTreeList - 1u)] = key[j];    // count of them
    } else if (l == 0) {
        sh.T[team] = base + lo;
        sh.need[team] = rank;
    }
    __syncthreads();
    if (bits > 0u)
#pragma unroll
        for (int j = 0; j < E; ++j) {
            if (!candidate(j)) continue;
            uint32_t gt = 0, eq = 0;
            for (uint32_t i = 0; i < count; ++i) {
                const uint32_t x = sh.list[team][i];
                gt += x > key[j] ? 1u : 0u;
                eq += x == key[j] ? 1u : 0u;
            }
            if (gt < rank && gt + eq >= rank) { sh.T[team] = key[j]; sh.need[team] = rank - gt; }     // (all who do agree)
        }
    __syncthreads();
    const uint32_t T = sh.T[team], need = sh.need[team];
    uint32_t mine = 0;                         // entries above T, and equal to it << 16
#pragma unroll
    for (int j = 0; j < E; ++j) {
        if (key[j] != kNoKey) mine += key[j] > T ? 1u : (key[j] == T ? 0x10000u : 0u);
    }
    const uint32_t incl = wave_incl_scan(mine);
    if (lane == kWave - 1) sh.wave[wave] = incl;
    __syncthreads();
    const uint32_t sums = row_incl_scan(lane < team_waves ? sh.wave[first_wave + lane] : 0u);
    const uint32_t w_in = wave - first_wave;
    const uint32_t before = incl - mine + (w_in ? lane_value(sums, w_in - 1u) : 0u);
    const uint32_t eq = before >> 16;
    return TeamCut{T, need, (before & 0xFFFFu) + (eq < need ? eq : need), eq};
}

// ---------------------------------------------------------------------------------
// speculative threshold of one worker in one block
// ---------------------------------------------------------------------------------

// Worker w = blockIdx.x.  Sample tile t covers [t*tile_stride, t*tile_stride + TILE) of the
// accumulated row (clipped to m), TILE lanes per tile; the block histograms the keys of all
// tiles in LDS and stores the lower edge of the bucket at which the count from the top
// reaches `target` (0 as in k_sample_pick).  It also clears the worker's candidate counter for the streaming pass
// that follows in stream order.  GENERAL, in front of the general kernels: blocks from P on clear
// what the rest of the step needs cleared (`job`), and a worker whose threshold is carried over
// (`carry`, see k_sample) takes that; BRACKET as in k_sample_pick, with samples as in k_sample (all values).  !SUM: the row is res alone, grad is not read.
template <int TILE, bool GENERAL, bool SUM, bool BRACKET = false>
__global__ __launch_bounds__(kSmallBlock) void k_small_sample(
        const float* __restrict__ grad, const float* __restrict__ res, uint32_t m, int64_t stride,
        uint32_t P, uint32_t tile_stride, uint32_t n_tiles, uint32_t target, uint32_t most, uint32_t* __restrict__ tspec,
        uint32_t* __restrict__ cand_count, const uint4* __restrict__ carry, ZeroJob job, uint32_t target_hi = 0u,
        uint32_t* __restrict__ thi = nullptr, uint32_t* __restrict__ samples = nullptr) {
    constexpr int kT = kSmallBlock;
    __shared__ uint32_t h[kSampleBins];
    __shared__ uint32_t s_wave[kT / kWave];
    __shared__ uint32_t s_out[3];
    const uint32_t t = threadIdx.x;
    if (GENERAL && blockIdx.x >= P) {
        const size_t step = (size_t)(gridDim.x - P) * kT, first = (size_t)(blockIdx.x - P) * kT + t;
#pragma unroll
        for (int a = 0; a < kZeroSlots; ++a)
            for (size_t i = first; i < job.n[a]; i += step) job.p[a][i] = 0u;
        return;
    }
    const int w = blockIdx.x;
    if (t == 0) cand_count[w] = 0u;
    if (GENERAL && carry) {
        const uint4 c = carry[w];
        if (c.x == 2u) {                             // block-uniform
            if (t == 0) tspec[w] = c.w;
            return;
        }
    }
    for (int b = t; b < kSampleBins; b += kT) h[b] = 0u;
    __syncthreads();
    const float* g = grad + (int64_t)w * stride;
    const float* r = res + (int64_t)w * stride;
    const uint32_t sub = t / TILE, el = t % TILE;
    constexpr uint32_t kTiles = kT / TILE;         // tiles the block takes side by side
    for (uint32_t t0 = sub; t0 < n_tiles; t0 += kTiles * kSmallSampleUnroll) {
        float gv[kSmallSampleUnroll], rv[kSmallSampleUnroll];
        bool ok[kSmallSampleUnroll];
#pragma unroll
        for (int u = 0; u < kSmallSampleUnroll; ++u) {
            const uint32_t tile = t0 + (uint32_t)u * kTiles;
            const uint64_t q = (uint64_t)tile * tile_stride + el;
            ok[u] = tile < n_tiles && q < m;
            gv[u] = SUM && ok[u] ? g[q] : 0.0f;
            rv[u] = ok[u] ? r[q] : 0.0f;
        }
        if (!SUM) {
            count_sampled(h, rv, ok);
            continue;
        }
#pragma unroll
        for (int u = 0; u < kSmallSampleUnroll; ++u) {
            const uint32_t bits = __float_as_uint(rv[u] + gv[u]);
            if (ok[u]) atomicAdd(&h[(bits & kAbs) >> kSampleShift], 1u);
            if (BRACKET && t0 + u * kTiles < n_tiles) {
                static_assert(!BRACKET || TILE == kSampleKept, "every sampled value is kept");
                samples[((size_t)w * n_tiles + t0 + u * kTiles) * kSampleKept + el] = ok[u] ? bits : 0xFFFFFFFFu;
            }
        }
    }
    __syncthreads();
    constexpr int kPer = kSampleBins / kT;
    uint32_t loc[kPer];
#pragma unroll
    for (int j = 0; j < kPer; ++j) loc[j] = h[t * kPer + j];
    suffix_pick<kPer>(loc, target, s_wave, s_out);
    if (t == 0) tspec[w] = s_out[2] && s_out[1] + s_out[2] <= most ? (s_out[0] << kSampleShift) : 0u;
    if (BRACKET) {
        if (t == 0) tspec[w] = upper_bound_key(tspec[w]);
        upper_end<kPer>(loc, target_hi, s_wave, s_out, thi + w);
    }
}

// ---------------------------------------------------------------------------------
// local selection of one worker in one block
// ---------------------------------------------------------------------------------

// The k largest of a whole row, for a worker whose candidate list cannot be used, by one block.  Every wave owns a part of
// the row, so that it counts and emits without a barrier; the row is read three times:
//   1. the first digit of all keys (bits 30 .. 19) is counted, the bin of the k-th key picked;
//   2. the keys in that bin go to a list in LDS, where a team selects; per wave the keys above it are counted.  A bin that
//      the list does not hold (masses of few magnitudes) is cut again before, unless its keys are all the same;
//   3. every wave emits its part.
// Bound by the latency of the one block's loads and by the instructions per key; a step with such rows, m = 524,288, P = 8,
// k = 2000, in us, by four to six walks of all waves in step / this: misled samples 706 / 180, zeros 166 / 146, ones 370 .. 472 / 193.
struct DenseShared {
    uint32_t h[kHistBins];                                     // the digits' counts, then the list
    uint32_t wave[kSmallBlock / kWave], out[3];
    uint32_t gt[kSmallBlock / kWave], eq[kSmallBlock / kWave]; // per wave: keys above the k-th, equal to it
    uint32_t n, ext[2], turn;
};
__device__ __forceinline__ uint32_t select_row(DenseShared& sh, TeamShared<1>& team, const float* __restrict__ row, uint32_t m, uint32_t k,
                                               uint32_t first_index, uint32_t* __restrict__ out_idx, float* __restrict__ out_val) {
    constexpr int kT = kSmallBlock, kWaves = kT / kWave, kU = 32;
    constexpr uint32_t kTurn = kWave * kU;
    const uint32_t t = threadIdx.x, lane = lane_id(), wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(t / kWave));
    const uint32_t turns = (m + kTurn - 1) / kTurn, per = (turns + kWaves - 1) / kWaves;
    const uint32_t first = wave * per, end = first + per < turns ? first + per : turns;
    // v[j]: element turn * kTurn + j * 64 + lane; behind the row zeros, which come after all of its own entries (k <= m)
    uint32_t v[kU];
    auto load = [&](uint32_t turn) {
        const uint32_t at = turn * kTurn;
        if (at + kTurn <= m) {
#pragma unroll
            for (int j = 0; j < kU; ++j) v[j] = __float_as_uint(row[at + j * kWave + lane]);
        } else {
#pragma unroll
            for (int j = 0; j < kU; ++j) {
                const uint32_t i = at + j * kWave + lane;
                const uint32_t x = __float_as_uint(row[i < m ? i : m - 1u]);
                v[j] = i < m ? x : 0u;
            }
        }
    };
    // adds 1 to h[b] for every lane with c (cm: their mask); masses of one key add once
    auto add = [&](bool c, uint64_t cm, uint32_t b) {
        const uint32_t b0 = lane_value(b, (uint32_t)__builtin_ctzll(cm));
        if (__ballot(c && b == b0) == cm) {
            if (lane == 0) atomicAdd(&sh.h[b0], (uint32_t)__popcll(cm));
        } else if (c) {
            atomicAdd(&sh.h[b], 1u);
        }
    };
    // whether the turn's keys are one: most of a row of zeros or of equal values
    auto one_key = [&]() {
        const uint32_t one = (uint32_t)__builtin_amdgcn_readfirstlane((int)(v[0] & kAbs));
        if (__ballot((v[0] & kAbs) != one || (v[kU - 1] & kAbs) != one) != 0ull) return false;
        uint32_t diff = 0;
#pragma unroll
        for (int j = 0; j < kU; ++j) diff |= v[j] ^ one;
        return __ballot((diff & kAbs) != 0u) == 0ull;
    };

    // ---- 1. first digit ----------------------------------------------------------------
    for (uint32_t b = t; b < (uint32_t)kHistBins; b += kT) sh.h[b] = 0u;
    __syncthreads();
    uint32_t run_bin = 0, run = 0;                             // wave-uniform: keys in steps that fell into one bin, not yet added
    auto flush = [&]() {
        if (lane == 0 && run) atomicAdd(&sh.h[run_bin], run);
    };
    for (uint32_t turn = first; turn < end; ++turn) {
        load(turn);
        if (one_key()) {
            flush();
            run_bin = (uint32_t)__builtin_amdgcn_readfirstlane((int)((v[0] & kAbs) >> kCoarseShift));
            run = kTurn;
            continue;
        }
#pragma unroll
        for (int j = 0; j < kU; ++j) {
            const uint32_t b = (v[j] & kAbs) >> kCoarseShift, b0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)b);
            if (__ballot(b != b0) != 0ull) {
                atomicAdd(&sh.h[b], 1u);
            } else {
                if (b0 != run_bin) {
                    flush();
                    run_bin = b0;
                    run = 0;
                }
                run += kWave;
            }
        }
    }
    flush();
    __syncthreads();
    uint32_t lo, bits = kCoarseShift, count, krem;             // the k-th key lies in [lo, lo + 2^bits), `count` keys do, its rank there
    {
        constexpr int kPer = kHistBins / kT;
        uint32_t loc[kPer];
#pragma unroll
        for (int j = 0; j < kPer; ++j) loc[j] = sh.h[t * kPer + j];
        suffix_pick<kPer>(loc, k, sh.wave, sh.out);
        lo = sh.out[0] << kCoarseShift;
        krem = k - sh.out[1];
        count = sh.out[2];
    }
    // ---- 2. the exact key --------------------------------------------------------------
    bool known = false;                                        // the per-wave counts are
    uint32_t T = 0, need = 0;
    while (count > (uint32_t)kHistBins && bits > 0u && !known) {         // block-uniform
        const uint32_t shift = bits > 11u ? bits - 11u : 0u, width = 1u << bits;
        __syncthreads();
        sh.h[t] = sh.h[t + kT] = 0u;
        if (t < 2) sh.ext[t] = 0u;
        __syncthreads();
        uint32_t gt = 0, in = 0, mx = 0, mn = kAbs;            // the first two wave-uniform
        for (uint32_t turn = first; turn < end; ++turn) {
            load(turn);
            if (one_key()) {
                const uint32_t key = (uint32_t)__builtin_amdgcn_readfirstlane((int)(v[0] & kAbs)), rel = key - lo;
                if (key < lo) continue;
                if (rel >= width) {
                    gt += kTurn;
                } else {
                    in += kTurn;
                    mx = key > mx ? key : mx;
                    mn = key < mn ? key : mn;
                    if (lane == 0) atomicAdd(&sh.h[rel >> shift], kTurn);
                }
                continue;
            }
#pragma unroll
            for (int j = 0; j < kU; ++j) {
                const uint32_t key = v[j] & kAbs, rel = key - lo;
                const uint64_t reach = __ballot(key >= lo);
                if (!reach) continue;
                const bool c = rel < width;
                const uint64_t cm = __ballot(c);
                gt += (uint32_t)__popcll(reach) - (uint32_t)__popcll(cm);
                if (!cm) continue;
                in += (uint32_t)__popcll(cm);
                if (c) {
                    mx = key > mx ? key : mx;
                    mn = key < mn ? key : mn;
                }
                add(c, cm, rel >> shift);
            }
        }
        mx = wave_largest(mx);
        mn = wave_largest(kAbs - mn);
        if (lane == 0) {
            atomicMax(&sh.ext[0], mx);
            atomicMax(&sh.ext[1], mn);
            sh.gt[wave] = gt;
            sh.eq[wave] = in;
        }
        __syncthreads();
        if (sh.ext[0] == kAbs - sh.ext[1]) {
            T = sh.ext[0];
            need = krem;
            known = true;
        } else {
            const uint32_t loc[2] = {sh.h[2 * t], sh.h[2 * t + 1]};
            suffix_pick<2>(loc, krem, sh.wave, sh.out);
            lo += sh.out[0] << shift;
            krem -= sh.out[1];
            count = sh.out[2];
            bits = shift;
        }
    }
    if (!known) {
        const uint32_t width = 1u << bits;
        __syncthreads();                                       // the picks have read h
        if (t == 0) sh.n = 0u;
        clear_teams(team);
        __syncthreads();
        uint32_t gt = 0, in = 0;                               // wave-uniform
        for (uint32_t turn = first; turn < end; ++turn) {
            load(turn);
#pragma unroll
            for (int j = 0; j < kU; ++j) {
                const uint32_t key = v[j] & kAbs, rel = key - lo;
                const uint64_t reach = __ballot(key >= lo);
                if (!reach) continue;
                const bool c = rel < width;
                const uint64_t cm = __ballot(c);
                gt += (uint32_t)__popcll(reach) - (uint32_t)__popcll(cm);
                if (!cm) continue;
                in += (uint32_t)__popcll(cm);
                if (bits == 0u) continue;
                uint32_t at = 0;
                if (lane == 0) at = atomicAdd(&sh.n, (uint32_t)__popcll(cm));
                at = lane_value(at, 0u) + rank_in(cm);
                if (c && at < (uint32_t)kHistBins) sh.h[at] = rel << 4 | wave;
            }
        }
        if (lane == 0) {
            sh.gt[wave] = gt;
            sh.eq[wave] = bits == 0u ? in : 0u;
        }
        __syncthreads();
        T = lo;
        need = krem;
        if (bits > 0u) {
            static_assert(kWaves <= 16 && kCoarseShift + 4 < 32, "a list entry's fields");
            constexpr int kPer = kHistBins / kT;
            const uint32_t n = sh.n < (uint32_t)kHistBins ? sh.n : (uint32_t)kHistBins;
            uint32_t key[kPer], owner[kPer];
#pragma unroll
            for (int j = 0; j < kPer; ++j) {
                const uint32_t e = sh.h[j * kT + t];
                key[j] = j * kT + t < n ? lo + (e >> 4) : kNoKey;
                owner[j] = e & 15u;
            }
            const TeamCut cut = team_select<kT>(team, key, lo, krem);
            T = cut.T;
            need = cut.need;
#pragma unroll
            for (int j = 0; j < kPer; ++j)
                if (key[j] != kNoKey && key[j] >= T) atomicAdd(key[j] > T ? &sh.gt[owner[j]] : &sh.eq[owner[j]], 1u);
            __syncthreads();
        }
    }
    // ---- 3. ordered emit ---------------------------------------------------------------
    const uint32_t gts = row_incl_scan(lane < (uint32_t)kWaves ? sh.gt[lane] : 0u), eqs = row_incl_scan(lane < (uint32_t)kWaves ? sh.eq[lane] : 0u);
    const uint32_t eq_end = lane_value(eqs, wave), gt_end = lane_value(gts, wave);
    uint32_t eq = wave ? lane_value(eqs, wave - 1u) : 0u;
    uint32_t out = (wave ? lane_value(gts, wave - 1u) : 0u) + (eq < need ? eq : need);
    const uint32_t out_end = gt_end + (eq_end < need ? eq_end : need);
    for (uint32_t turn = first; turn < end && out < out_end; ++turn) {
        load(turn);
#pragma unroll
        for (int j = 0; j < kU; ++j) {
            const uint32_t key = v[j] & kAbs;
            if (__ballot(key >= T) == 0ull) continue;
            const uint64_t eqm = __ballot(key == T);
            const bool sel = key > T || (key == T && eq + rank_in(eqm) < need);
            const uint64_t sm = __ballot(sel);
            const uint32_t i = turn * kTurn + j * kWave + lane, pos = out + rank_in(sm);
            if (sel && pos < k && i < m) {                     // (always so)
                out_idx[pos] = first_index + i;
                out_val[pos] = __uint_as_float(v[j]);
            }
            out += (uint32_t)__popcll(sm);
            eq += (uint32_t)__popcll(eqm);
        }
    }
    return T;
}

// The k largest of the entries that a block's threads hold in index order, E each (key kNoKey: none); k of them reach `bound`.
// Returns the k-th key.
template <int E>
__device__ __forceinline__ uint32_t select_held(TeamShared<1>& team, const uint32_t (&idx)[E], const uint32_t (&bits)[E],
                                                const uint32_t (&key)[E], uint32_t bound, uint32_t k, uint32_t* __restrict__ out_idx,
                                                float* __restrict__ out_val) {
    const TeamCut cut = team_select<(uint32_t)kSmallBlock>(team, key, bound, k);
    uint32_t eq = cut.eq, pos = cut.pos;
#pragma unroll
    for (int c = 0; c < E; ++c) {
        if (key[c] == kNoKey) continue;
        bool sel = key[c] > cut.T;
        if (key[c] == cut.T) sel = eq++ < cut.need;
        if (sel && pos < k) {                                  // (always inside)
            out_idx[pos] = idx[c];
            out_val[pos] = __uint_as_float(bits[c]);
            ++pos;
        }
    }
    return cut.T;
}

// Worker s = blockIdx.x.  The items are the worker's candidate list, or, if the
// speculative threshold left fewer than k candidates or more than the list holds, its
// dense row (select_row).  A candidate list of at most
// 1024 E entries is held in registers and selected from by the block as one team, as few entries per thread as the list
// takes (gtopk_local_select in us, E entries for the first threads, loaded one after the other / this: m = 400,000, P = 4, k = 4000
// 45 / 38; m = 200,000, P = 8, k = 2000 46 / 37, three kernels 41; m = 524,288, P = 1, k = 1000 33 / 29).  A longer one takes
// three stages, each a walk over it:
//   1. LDS histogram of the first digit -> the bin d1 of the k-th key;
//   2. up to three LDS radix passes over the keys inside bin d1 -> the exact key T and the
//      number of ties to take;
//   3. the emit in index order, run after run in chunk order.
// Blocks (s, 1) .. share the row of a worker that has to be read whole, gridDim.y * k <= 1024 kRowPart, and return at once
// from any other (arrived: a word per worker, zero; no block waits for another).
// E: entries of a candidate list that a thread holds.  T_out != NULL: the smallest key of each set, for what follows in
// the general path (where thresholds are carried on as well).
template <int E>
__global__ __launch_bounds__(kSmallBlock) void k_small_select(
        CandSrc src, uint32_t k, uint32_t* __restrict__ out_idx, float* __restrict__ out_val, uint32_t* __restrict__ T_out,
        uint32_t* __restrict__ arrived) {
    constexpr int kT = kSmallBlock;
    __shared__ DenseShared sh;
    __shared__ uint32_t s_rx[kSmallMaxChunks];
    __shared__ uint32_t s_roff[kSmallMaxChunks + 1];
    __shared__ TeamShared<1> s_team;
    uint32_t* h = sh.h;
    uint32_t* s_wave = sh.wave;
    uint32_t* s_out = sh.out;
    const int s = blockIdx.x;
    const uint32_t t = threadIdx.x;
    if (src.dense(s)) {                                        // block-uniform
        const float* row = src.res + (int64_t)s * src.stride;
        uint32_t T;
        if (gridDim.y == 1u) {
            T = select_row(sh, s_team, row, src.m, k, 0u, out_idx + (size_t)s * k, out_val + (size_t)s * k);
        } else {
            // every block selects k entries of its part of the row; the last to be done selects among those
            const uint32_t len = ((src.m + gridDim.y - 1u) / gridDim.y + 1023u) & ~1023u, first = blockIdx.y * len;
            const size_t part = (size_t)s * src.cap + (size_t)blockIdx.y * k;
            uint32_t* bounds = src.run_off + (size_t)s * src.nchunks;        // (not in use here, as the ordered list is not)
            T = select_row(sh, s_team, row + first, src.m - first < len ? src.m - first : len, k, first, src.ord_idx + part,
                           src.ord_val + part);
            if (t == 0) bounds[blockIdx.y] = T;
            // (every wave's stores have reached the L2 before the block meets; then one fence writes them back for the last
            // block, which may sit on another XCD)
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
            if (t == 0) {
                __threadfence();
                sh.turn = atomicAdd(&arrived[s], 1u);
            }
            clear_teams(s_team);
            __syncthreads();
            if (sh.turn != gridDim.y - 1u) return;             // block-uniform
            __threadfence();
            const uint32_t n = gridDim.y * k;                  // <= 1024 kRowPart
            uint32_t idx[kRowPart], bits[kRowPart], key[kRowPart], bound = 0;
            for (uint32_t y = 0; y < gridDim.y; ++y) bound = op_max(bound, bounds[y]);
#pragma unroll
            for (int c = 0; c < kRowPart; ++c) {
                const uint32_t e = t * kRowPart + c;
                const size_t at = (size_t)s * src.cap + (e < n ? e : 0u);
                idx[c] = src.ord_idx[at];
                bits[c] = __float_as_uint(src.ord_val[at]);
                key[c] = e < n ? bits[c] & kAbs : kNoKey;
            }
            T = select_held(s_team, idx, bits, key, bound, k, out_idx + (size_t)s * k, out_val + (size_t)s * k);
        }
        if (T_out && t == 0) {
            T_out[s] = T;
            src.carry(s, T);
        }
        return;
    }
    if (blockIdx.y != 0u) return;
    const uint32_t n = src.nphys(s, false);
    if (n <= (uint32_t)(E * kT)) {
        // ---- a short candidate list: every thread takes E consecutive entries in index order (run after run in
        // chunk order); the block selects the k largest, ties to the lower index (Algorithm 4 line 5)
        const uint32_t nruns = src.nchunks;                    // <= kSmallMaxChunks <= kT
        uint2 run = make_uint2(0u, 0u);
        if (t < nruns) run = src.run_table[(size_t)s * src.nchunks + t];
        clear_teams(s_team);
        uint32_t tot;
        const uint32_t incl = block_incl_scan(run.y, s_wave, tot);
        if (t < nruns) { s_rx[t] = run.x; s_roff[t + 1] = incl; }
        if (t == 0) s_roff[0] = 0u;
        __syncthreads();
        // (as few entries per thread as the list takes, so that all waves share it; their loads in flight together)
        const uint32_t ept = (n + kT - 1) / kT;                // <= E
        const uint32_t entry = t * ept < n ? t * ept : n - 1u; // (k <= n; a thread without any entry repeats the last)
        uint32_t idx[E], bits[E], key[E];
        uint32_t r = 0;
        {
            uint32_t hi = nruns;                               // the run r with roff[r] <= entry < roff[r+1]
            while (hi - r > 1) {
                const uint32_t mid = (r + hi) >> 1;
                if (s_roff[mid] <= entry) r = mid; else hi = mid;
            }
        }
#pragma unroll
        for (int c = 0; c < E; ++c) {
            idx[c] = 0u; bits[c] = 0u;
            if ((uint32_t)c < ept) {                           // block-uniform
                const uint32_t lp = entry + c < n ? entry + c : n - 1u;
                while (s_roff[r + 1] <= lp) ++r;               // (r + 1 <= nruns: the last run ends at n)
                src.fetch_phys(s, false, s_rx[r] + (lp - s_roff[r]), idx[c], bits[c]);
            }
        }
#pragma unroll
        for (int c = 0; c < E; ++c) key[c] = (uint32_t)c < ept && t * ept + c < n ? bits[c] & kAbs : kNoKey;
        const uint32_t T = select_held(s_team, idx, bits, key, src.tspec[s], k, out_idx + (size_t)s * k, out_val + (size_t)s * k);
        if (T_out && t == 0) {
            T_out[s] = T;
            src.carry(s, T);
        }
        return;
    }
    constexpr int kAhead = 16;                                 // loads in flight per thread
    const uint32_t first = t / kWave * (kWave * kAhead) + lane_id();          // a wave's keys of a turn lie next to each other
    const Digit dg = src.digit(s, false, SelState{});

    // ---- 1. first digit --------------------------------------------------------------
    for (int b = t; b < kHistBins; b += kT) h[b] = 0u;
    __syncthreads();
    for (uint32_t p0 = 0; p0 < n; p0 += kT * kAhead) {
        if (p0 + (first - lane_id()) >= n) break;
        uint32_t key[kAhead];
        bool ok[kAhead];
#pragma unroll
        for (int j = 0; j < kAhead; ++j) {
            const uint32_t p = p0 + first + j * kWave;
            src.fetch_key_phys(s, false, p < n ? p : n - 1, key[j]);
        }
#pragma unroll
        for (int j = 0; j < kAhead; ++j) ok[j] = p0 + first + j * kWave < n;
#pragma unroll
        for (int j = 0; j < kAhead; ++j) {
            // a wave whose keys all fall into one bin (equal values) adds once
            const uint32_t b = dg.bin(key[j]);
            const uint64_t act = __ballot(ok[j]);
            if (act == 0) continue;
            const uint32_t b0 = lane_value(b, (uint32_t)__builtin_ctzll(act));
            if (__ballot(ok[j] && b == b0) == act) {
                if (lane_id() == (uint32_t)__builtin_ctzll(act)) atomicAdd(&h[b0], (uint32_t)__popcll(act));
            } else if (ok[j]) {
                atomicAdd(&h[b], 1u);
            }
        }
    }
    __syncthreads();
    uint32_t d1, krem;
    {
        constexpr int kPer = kHistBins / kT;
        uint32_t loc[kPer];
#pragma unroll
        for (int j = 0; j < kPer; ++j) loc[j] = h[t * kPer + j];
        suffix_pick<kPer>(loc, k, s_wave, s_out);
        d1 = s_out[0];
        krem = k - s_out[1];
    }
    // ---- 2. the exact key --------------------------------------------------------------
    const uint32_t lo = dg.lo(d1), width = dg.width(d1);    // bin d1 = [lo, lo + width)
    uint32_t prefix = 0;          // value of the rel bits above the current pass
    for (int pass = 0; pass < 3; ++pass) {
        const int shift = pass == 0 ? 20 : (pass == 1 ? 10 : 0);
        const int bits = pass == 0 ? 11 : 10;
        if (shift > 0 && width <= (1u << shift)) continue;       // uniform
        __syncthreads();                                         // the last pick has read h
        for (int b = t; b < 2048; b += kT) h[b] = 0u;
        __syncthreads();
        for (uint32_t p0 = 0; p0 < n; p0 += kT * kAhead) {
            if (p0 + (first - lane_id()) >= n) break;
            uint32_t key[kAhead];
            bool ok[kAhead];
#pragma unroll
            for (int j = 0; j < kAhead; ++j) {
                const uint32_t p = p0 + first + j * kWave;
                src.fetch_key_phys(s, false, p < n ? p : n - 1, key[j]);
            }
#pragma unroll
            for (int j = 0; j < kAhead; ++j) ok[j] = p0 + first + j * kWave < n;
#pragma unroll
            for (int j = 0; j < kAhead; ++j) {
                const uint32_t rel = key[j] - lo;
                const bool mine = ok[j] && dg.bin(key[j]) == d1 && (rel >> (shift + bits)) == prefix;
                const uint32_t b = (rel >> shift) & ((1u << bits) - 1u);
                const uint64_t act = __ballot(mine);
                if (act == 0) continue;
                const uint32_t b0 = lane_value(b, (uint32_t)__builtin_ctzll(act));
                if (__ballot(mine && b == b0) == act) {
                    if (lane_id() == (uint32_t)__builtin_ctzll(act)) atomicAdd(&h[b0], (uint32_t)__popcll(act));
                } else if (mine) {
                    atomicAdd(&h[b], 1u);
                }
            }
        }
        __syncthreads();
        const uint32_t loc[2] = {h[2 * t], h[2 * t + 1]};
        suffix_pick<2>(loc, krem, s_wave, s_out);
        prefix = (prefix << bits) | s_out[0];
        krem -= s_out[1];
    }
    const uint32_t T = lo + prefix;
    const uint32_t need = krem;
    if (T_out && t == 0) {
        T_out[s] = T;
        src.carry(s, T);
    }

    // ---- 3. ordered emit ---------------------------------------------------------------
    // the list is read run after run in chunk order: first slots and running counts
    const uint32_t nruns = src.nchunks;                        // <= kSmallMaxChunks <= kT
    uint2 run = make_uint2(0u, 0u);
    if (t < nruns) run = src.run_table[(size_t)s * src.nchunks + t];
    uint32_t tot;
    const uint32_t incl = block_incl_scan(run.y, s_wave, tot);
    if (t < nruns) { s_rx[t] = run.x; s_roff[t + 1] = incl; }
    if (t == 0) s_roff[0] = 0u;
    __syncthreads();
    // eight consecutive entries per thread and turn, one prefix sum; the rest of the list behind the k-th entry is not read
    constexpr uint32_t kTurn = 8;
    uint32_t gt_before = 0, eq_before = 0;
    for (uint32_t base = 0; base < n; base += kT * kTurn) {
        const uint32_t lp0 = base + t * kTurn;
        uint32_t r = 0;
        if (lp0 < n) {
            uint32_t hi = nruns;                        // the run r with roff[r] <= lp0 < roff[r+1]
            while (hi - r > 1) {
                const uint32_t mid = (r + hi) >> 1;
                if (s_roff[mid] <= lp0) r = mid; else hi = mid;
            }
        }
        uint32_t idx[kTurn], bits[kTurn], key[kTurn], mine = 0;         // entries above T, and equal to it << 16
#pragma unroll
        for (uint32_t j = 0; j < kTurn; ++j) {
            const uint32_t lp = lp0 + j < n ? lp0 + j : n - 1;
            while (s_roff[r + 1] <= lp) ++r;
            src.fetch_phys(s, false, s_rx[r] + (lp - s_roff[r]), idx[j], bits[j]);
        }
#pragma unroll
        for (uint32_t j = 0; j < kTurn; ++j) {
            key[j] = bits[j] & kAbs;
            if (lp0 + j >= n) key[j] = kNoKey;
            if (key[j] != kNoKey) mine += key[j] > T ? 1u : (key[j] == T ? 0x10000u : 0u);
        }
        uint32_t all;
        const uint32_t before = block_incl_scan(mine, s_wave, all) - mine;
        uint32_t eq = eq_before + (before >> 16), pos = gt_before + (before & 0xFFFFu) + (eq < need ? eq : need);
#pragma unroll
        for (uint32_t j = 0; j < kTurn; ++j) {
            if (key[j] == kNoKey) continue;
            bool sel = key[j] > T;
            if (key[j] == T) sel = eq++ < need;
            if (sel && pos < k) {       // always inside when the counts are consistent
                out_idx[(size_t)s * k + pos] = idx[j];
                out_val[(size_t)s * k + pos] = __uint_as_float(bits[j]);
                ++pos;
            }
        }
        gt_before += all & 0xFFFFu;
        eq_before += all >> 16;
        if (gt_before + (eq_before < need ? eq_before : need) >= k) break;                    // block-uniform
    }
}

// ---------------------------------------------------------------------------------
// the whole tree, the average and the extra residual in one block
// ---------------------------------------------------------------------------------

// All P k-sets sit in LDS (P * k <= 4096 entries).  Round j merges set 2p with set 2p+1 of the surviving sets for
// every pair p, the pairs side by side: a wave each where the sets are short (tree_round_by_waves), else a team of
// 1024 / pairs threads (at most 8 pairs, as sets of more than 128 entries come 31 at most), of which a thread owns at most
// kTreeEpt consecutive slots of its pair's union in index order:
//   union      a binary search along the diagonal, then a sequential merge; A's copy carries the sum at a shared
//              index, B's slot there is a tombstone;
//   select     see team_select; the larger of the operands' smallest keys is the bound, which k keys reach unless sums cancel;
//   emit       one prefix sum over the team's threads, selected slots to set p of the next round.
// (Every barrier is the block's, about nine per round, and a round is its chain of dependent LDS reads and barriers:
// some 6 us.  One wave per pair that held all keys in registers and searched the k-th in a bracket, with the slots in
// LDS for a bitmap and a compaction, took 8 us per round of sets of 270; the tree of 8 such sets 26.9 -> 20.0 us, the selection
// of 270 among 680 candidates 10.6 -> 7.5.)
// After the last round the global set's values are divided by P and written out, and every worker's locally selected
// entries whose index is in it (or whose value is -0.0, which the literal zero-then-add-back would turn into +0.0) are
// stored as +0.0 in the worker's row - the rows still hold the accumulated values at the selected entries.
struct TreeShared {
    // two buffers of surviving sets, k entries each, that the rounds take in turn
    uint32_t idx[kSmallMaxEntries + kSmallMaxEntries / 2];
    uint32_t val[kSmallMaxEntries + kSmallMaxEntries / 2];
    TeamShared<kTreeTeams> team;
    uint32_t min[2][kSmallMaxP];                               // the sets' smallest keys
};

// Slots [l * ept, (l + 1) * ept) of the union of pair q, in index order (ept <= E): kTomb where there is none.
template <int E>
__device__ __forceinline__ void tree_union(const TreeShared& sh, uint32_t q, uint32_t k, uint32_t from, uint32_t l, uint32_t ept,
                                           uint32_t (&oi)[E], uint32_t (&ov)[E]) {
    const uint32_t n = 2 * k;
    const uint32_t* ai = sh.idx + from + 2 * q * k;
    const uint32_t* bi = ai + k;
    const uint32_t* av = sh.val + from + 2 * q * k;
    const uint32_t* bv = av + k;
#pragma unroll
    for (int j = 0; j < E; ++j) { oi[j] = kTomb; ov[j] = 0u; }
    const uint32_t d0 = l * ept;
    if (d0 < n) {
        uint32_t x = d0 > k ? d0 - k : 0u, hi = d0 < k ? d0 : k;
        while (x < hi) {
            const uint32_t mid = (x + hi) >> 1;
            if (ai[mid] <= bi[d0 - 1 - mid]) x = mid + 1; else hi = mid;
        }
        uint32_t y = d0 - x;
        uint32_t a = x < k ? ai[x] : kTomb, b = y < k ? bi[y] : kTomb, aprev = x > 0 ? ai[x - 1] : kTomb;
#pragma unroll
        for (int j = 0; j < E; ++j) {
            if ((uint32_t)j >= ept || d0 + j >= n) continue;
            if (a <= b && x < k) {
                oi[j] = a;
                ov[j] = av[x];
                if (b == a) ov[j] = __float_as_uint(__uint_as_float(ov[j]) + __uint_as_float(bv[y]));   // one fp32 add
                aprev = a;
                ++x;
                a = x < k ? ai[x] : kTomb;
            } else if (y < k) {
                oi[j] = b == aprev ? kTomb : b;
                ov[j] = bv[y];
                ++y;
                b = y < k ? bi[y] : kTomb;
            }
        }
    }
}

// One round, SIZE threads per team and a pair per team: the sets at `from` are merged into those at `to`.
template <uint32_t SIZE>
__device__ __forceinline__ void tree_round(TreeShared& sh, uint32_t k, uint32_t from, uint32_t to, int turn_min) {
    const uint32_t q = threadIdx.x / SIZE, l = threadIdx.x % SIZE;            // the team's pair
    constexpr int kE = SIZE == 1024 ? 1 : (SIZE == 512 ? 2 : kTreeEpt);       // slots per thread, at most
    static_assert(2 * kSmallMaxK <= 1024 && kSmallMaxEntries <= 1024 * kTreeEpt, "2k slots fit a team's threads");
    const uint32_t n = 2 * k, ept = (n + SIZE - 1) / SIZE;                   // <= kE
    const uint32_t bound = op_max(sh.min[turn_min][2 * q], sh.min[turn_min][2 * q + 1]);
    uint32_t oi[kE], ov[kE];
    tree_union<kE>(sh, q, k, from, l, ept, oi, ov);
    // ---- select and emit ------------------------------------------------------------
    uint32_t key[kE];
#pragma unroll
    for (int j = 0; j < kE; ++j) key[j] = oi[j] != kTomb ? ov[j] & kAbs : kNoKey;
    const TeamCut c = team_select<SIZE>(sh.team, key, bound, k);
    if (l == 0) sh.min[turn_min ^ 1][q] = c.T;
    uint32_t eq = c.eq, pos = c.pos;
#pragma unroll
    for (int j = 0; j < kE; ++j) {
        if (key[j] == kNoKey) continue;
        bool sel = key[j] > c.T;
        if (key[j] == c.T) sel = eq++ < c.need;
        if (sel && pos < k) {                  // (always inside)
            sh.idx[to + q * k + pos] = oi[j];
            sh.val[to + q * k + pos] = ov[j];
            ++pos;
        }
    }
    __syncthreads();
}

// One round of sets of at most 32 E entries, a wave per pair and 2 E slots per lane at most, no barrier but the one at
// the end: for sets this short the teams' barriers are most of a round.  The k-th key is found bit by bit, the keys of all
// lanes counted by ballots; most searches end early, with a bound that exactly k keys reach.  A step at m = 20,000 in us, by
// a wave per pair that searched in a bracket / by teams / this:  P = 64  k = 1   43.3 / 50.3 / 28.8   k = 32   48.8 / 57.8 / 36.9
// P = 16  k = 8   34.0 / 37.1 / 26.9   k = 128  46.8 / 41.3 / 36.3   P = 4  k = 32   27.1 / 27.1 / 23.4   k = 128  32.7 / 28.3 / 26.8
template <int E>
__device__ __forceinline__ void tree_round_by_waves(TreeShared& sh, uint32_t pairs, uint32_t k, uint32_t from, uint32_t to, int turn_min) {
    const uint32_t lane = lane_id(), wave = threadIdx.x / kWave;
    for (uint32_t q = wave; q < pairs; q += kSmallBlock / kWave) {           // wave-uniform
        uint32_t oi[E], ov[E], key[E];
        tree_union<E>(sh, q, k, from, lane, (2 * k + kWave - 1) / kWave, oi, ov);
#pragma unroll
        for (int j = 0; j < E; ++j) key[j] = oi[j] != kTomb ? ov[j] & kAbs : kNoKey;
        // a bound that k keys reach: the larger of the operands' smallest keys, unless sums cancel
        auto reach = [&](uint32_t least) {                   // (never kNoKey; none reach a least above kAbs, which the search may try)
            uint32_t n = 0;
#pragma unroll
            for (int j = 0; j < E; ++j) n += (uint32_t)__popcll(__ballot(key[j] + 1u > least));
            return n;
        };
        uint32_t base = op_max(sh.min[turn_min][2 * q], sh.min[turn_min][2 * q + 1]);
        base = (uint32_t)__builtin_amdgcn_readfirstlane((int)base);
        uint32_t n = reach(base);
        if (n < k) {
            base = 0u;
            n = reach(0u);
        }
        uint32_t most = 0;
#pragma unroll
        for (int j = 0; j < E; ++j) most = key[j] != kNoKey && key[j] > most ? key[j] : most;
        most = wave_largest(most);
        uint32_t T = base;                                   // n keys reach T, at least k
        if (n > k && most > base) {
            for (int b = 31 - __builtin_clz(most - base); b >= 0 && n != k; --b) {
                const uint32_t c = reach(T + (1u << b));
                if (c >= k) {
                    T += 1u << b;
                    n = c;
                }
            }
        }
        uint32_t ties = 0xFFFFFFFFu;                         // keys equal to T to take
        if (n == k) {                                        // those that reach T, all of them: T becomes the smallest
            uint32_t inv = 0;
#pragma unroll
            for (int j = 0; j < E; ++j) inv = key[j] - T <= kAbs - T ? op_max(inv, kAbs - key[j]) : inv;
            T = kAbs - wave_largest(inv);
        } else if (n > k) {
            ties = k - reach(T + 1u);
        }
        if (lane == 0) sh.min[turn_min ^ 1][q] = T;
        // (slots lane by lane: those of the lanes below first)
        uint32_t eq = 0, pos = 0, mine = 0;                  // mine: selected for certain, and equal to T << 16
#pragma unroll
        for (int j = 0; j < E; ++j)
            if (key[j] != kNoKey) mine += key[j] > T ? 1u : (key[j] == T ? 0x10000u : 0u);
        const uint32_t before = wave_incl_scan(mine) - mine;
        eq = before >> 16;
        pos = (before & 0xFFFFu) + (eq < ties ? eq : ties);
#pragma unroll
        for (int j = 0; j < E; ++j) {
            if (key[j] == kNoKey) continue;
            bool sel = key[j] > T;
            if (key[j] == T) sel = eq++ < ties;
            if (sel && pos < k) {                            // (always inside)
                sh.idx[to + q * k + pos] = oi[j];
                sh.val[to + q * k + pos] = ov[j];
                ++pos;
            }
        }
    }
    __syncthreads();
}

// E: 0: teams of threads (sets of more than 128 entries); else waves (sets of at most 32 E entries).
// (The teams' four sizes in one kernel take 128 registers and spill three; with the sizes known only at run time the tree of 8
// sets of 270 takes 23.4 us instead of 20.)
template <int E>
__global__ __launch_bounds__(kSmallBlock) void k_small_tree(
        const uint32_t* __restrict__ loc_idx, const float* __restrict__ loc_val, uint32_t P,
        uint32_t k, uint32_t* __restrict__ g_idx, float* __restrict__ g_val, float divisor,
        float* __restrict__ res, int64_t stride) {
    constexpr int kT = kSmallBlock;
    constexpr int kWaves = kT / kWave;
    constexpr int kPer = kSmallMaxEntries / kT;       // entries of the input sets per thread
    __shared__ TreeShared sh;
    const uint32_t t = threadIdx.x, lane = lane_id(), wave = t / kWave;
    const uint32_t total = P * k;
    uint32_t in_idx[kPer], in_val[kPer];              // kept for the extra residual
#pragma unroll
    for (int c = 0; c < kPer; ++c) {
        const uint32_t e = (uint32_t)c * kT + t;
        in_idx[c] = 0u; in_val[c] = 0u;
        if (e < total) {
            in_idx[c] = loc_idx[e];
            in_val[c] = __float_as_uint(loc_val[e]);
            sh.idx[e] = in_idx[c];
            sh.val[e] = in_val[c];
        }
    }
    clear_teams(sh.team);
    __syncthreads();
    for (uint32_t w = wave; w < P; w += kWaves) {      // smallest keys, a wave per set
        uint32_t inv = 0;
        for (uint32_t x = lane; x < k; x += kWave) inv = op_max(inv, kAbs - (sh.val[w * k + x] & kAbs));
        inv = wave_largest(inv);
        if (lane == 0) sh.min[0][w] = kAbs - inv;
    }
    __syncthreads();
    uint32_t from = 0, to = kSmallMaxEntries;         // the buffers
    int turn_min = 0;
    for (uint32_t nsets = P; nsets > 1; nsets >>= 1) {
        const uint32_t pairs = nsets >> 1;
        if constexpr (E != 0) tree_round_by_waves<E>(sh, pairs, k, from, to, turn_min);
        else if (pairs == 1) tree_round<1024>(sh, k, from, to, turn_min);
        else if (pairs == 2) tree_round<512>(sh, k, from, to, turn_min);
        else if (pairs == 4) tree_round<256>(sh, k, from, to, turn_min);
        else tree_round<128>(sh, k, from, to, turn_min);
        const uint32_t x = from;
        from = to;
        to = x;
        turn_min ^= 1;
    }
    const uint32_t* a_idx = sh.idx + from;              // the global set
    const uint32_t* a_val = sh.val + from;
    // ---- the global set: average, write out ------------------------------------------------
    for (uint32_t i = t; i < k; i += kT) {
        g_idx[i] = a_idx[i];
        g_val[i] = __uint_as_float(a_val[i]) / divisor;
    }
    // ---- extra residual ---------------------------------------------------------------------
    if (res) {
#pragma unroll
        for (int c = 0; c < kPer; ++c) {
            const uint32_t e = (uint32_t)c * kT + t;
            if (e >= total) break;
            const uint32_t w = e / k;
            const uint32_t i = in_idx[c];
            uint32_t lo = 0, hi = k;
            while (lo < hi) { const uint32_t mid = (lo + hi) >> 1; if (a_idx[mid] < i) lo = mid + 1; else hi = mid; }
            const bool in_g = lo < k && a_idx[lo] == i;
            if (in_g || in_val[c] == 0x80000000u) res[(int64_t)w * stride + i] = 0.0f;
        }
    }
}

}  // namespace gtopk
